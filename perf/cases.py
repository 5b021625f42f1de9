"""The work that users of this package have it do, as timed cases.

Six kinds, each through the public entry points of `binding` and `rollout`:

  rollout          one block denoised to completion with GpuRollout.run_block: cache refresh, then attention, LM head
                   and commit per step until nothing is masked (the serving / RL-rollout path)
  step             one denoising step through the binding's own calls, for callers with a loop of their own; the cached
                   prefixes of the batch may be ragged
  varlen_train     attention over a packed batch of unequal sequences, forward and backward (SFT, actor update)
  diffusion_train  block-diffusion training attention over the pair (noisy, clean), forward and backward of both halves
  logprob          masked log-likelihood of given responses: LM head with targets, summed per sequence
  full_pass        one full-sequence block-causal pass: attention, LM head over the masked rows, one commit per block

Sizes are those of the workloads in `synth`, of the tests and of the benchmark; weights are N(0, Dh^-1/2) and activations
N(0, 1) as there, so that confident and unconfident positions both occur.
"""
import math

import torch

from paper_2604_04215_amd import binding as dlm
from paper_2604_04215_amd.rollout import GpuRollout
from paper_2604_04215_amd.synth import Config

BF16, F32, I32, U8 = torch.bfloat16, torch.float32, torch.int32, torch.uint8
DEV = "cuda:0"


# --------------------------------------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------------------------------------
def _rollout(B, Hq, Hkv, d, Dh, V, prompt, blocks_before, blocks_after, Lb, rule, tau=0.9, k=0, dual=False, bs=0, masked=0, refresh=True,
             sampled=False, confidence="prob"):
    """blocks_before / blocks_after: blocks of the response in front of and behind the one being denoised; bs: block size of the block-causal mask
    (0: every position sees every other); masked: positions masked at the start (0: all of them)."""
    return dict(kind="rollout", B=B, Hq=Hq, Hkv=Hkv, d=d, Dh=Dh, V=V, prompt=prompt, blocks_before=blocks_before, blocks_after=blocks_after, Lb=Lb,
                rule=rule, tau=tau, k=k, dual=dual, bs=bs, masked=masked, refresh=refresh, sampled=sampled, confidence=confidence)


def _step(B, Hq, Hkv, d, Dh, V, prefix, Lb, k, ragged):
    return dict(kind="step", B=B, Hq=Hq, Hkv=Hkv, d=d, Dh=Dh, V=V, prefix=prefix, Lb=Lb, k=k, ragged=ragged)


def _varlen(B, Hq, Hkv, d, prompt_lo, prompt_hi, resp_lo, resp_hi, bs=0):
    return dict(kind="varlen_train", B=B, Hq=Hq, Hkv=Hkv, d=d, prompt_lo=prompt_lo, prompt_hi=prompt_hi, resp_lo=resp_lo, resp_hi=resp_hi, bs=bs)


def _diffusion(B, L, Hq, Hkv, d, bs):
    return dict(kind="diffusion_train", B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, bs=bs)


def _logprob(B, n_pos, Dh, V, mask_prob):
    return dict(kind="logprob", B=B, n_pos=n_pos, Dh=Dh, V=V, mask_prob=mask_prob)


def _full(B, L, Hq, Hkv, d, Dh, V, bs):
    return dict(kind="full_pass", B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, Dh=Dh, V=V, bs=bs)


def listed():
    return [
        # the smallest problem of the test and benchmark workloads: twenty-odd microseconds of kernels per step, so launches, the host
        # loop and every kernel's fixed latency are what counts
        dict(_rollout(1, 4, 4, 64, 256, 2048, 256, 0, 0, 32, "threshold", masked=16, refresh=False), name="rollout_tiny"),
        # interactive use: one sequence with a long context, one step of the fixed schedule (2 tokens a step)
        dict(_step(1, 32, 8, 128, 4096, 157184, 8192, 32, 2, False), name="step_single_long"),
        # the benchmark's default: 8B-class multi-head rollout of a group of 8, a block in the middle of the response
        dict(_rollout(8, 32, 32, 128, 4096, 126464, 512, 4, 0, 32, "threshold"), name="rollout_mha"),
        # the same model with the dual cache: the block sees the still masked blocks behind it, twice the batch, longer context
        dict(_rollout(16, 32, 32, 128, 4096, 126464, 1024, 7, 8, 32, "threshold", dual=True), name="rollout_dual"),
        # 7B-class grouped-query model, fixed number of commits per step, a large batch: the LM head is a real matrix product here
        dict(_rollout(32, 28, 4, 128, 3584, 152064, 768, 3, 0, 32, "topk", k=4), name="rollout_gqa_topk"),
        # block-diffusion model: blocks of 4 at the end of a 4096-token sequence, 64 sequences, a gigabyte of cache
        dict(_rollout(64, 32, 8, 128, 4096, 157184, 4092, 0, 0, 4, "threshold", tau=0.95, bs=4), name="rollout_block_causal"),
        # RL group of 8 sampled rollouts of one odd-sized prompt, fixed schedule of 2 tokens a step
        dict(_rollout(8, 28, 4, 128, 3584, 152064, 391, 2, 0, 32, "topk", k=2, sampled=True), name="rollout_sampled"),
        # SFT / actor update: 128 packed sequences (64 k tokens), multi-head, bidirectional
        dict(_varlen(128, 32, 32, 128, 64, 384, 32, 512), name="varlen_train_mha"),
        # a small ragged batch of the same kind, block-causal, grouped-query, head size 64
        dict(_varlen(24, 14, 2, 64, 1, 200, 0, 333, bs=32), name="varlen_train_small"),
        # block-diffusion training: noisy and clean copy of 8 sequences of 4096 tokens in blocks of 4
        dict(_diffusion(8, 4096, 32, 8, 128, 4), name="diffusion_train"),
        # old-policy / reference log-probabilities of a group of 16 responses of up to 512 tokens, half of them masked
        dict(_logprob(16, 512, 4096, 126464, 0.5), name="logprob_group"),
        # the full-sequence training-style pass at its full size: 262 144 tokens, half of them through the LM head
        dict(_full(64, 4096, 32, 8, 128, 4096, 157184, 4), name="full_pass"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(4, 4, 64), (14, 2, 64), (32, 32, 128), (28, 4, 128), (32, 8, 128), (16, 2, 128)]
_DH = [256, 1024, 2048, 3584, 4096]


def draw(rng):
    kind = rng.choice(["rollout", "rollout", "rollout", "step", "varlen_train", "diffusion_train", "logprob", "full_pass"])
    Hq, Hkv, d = rng.choice(_HEADS)
    Dh = rng.choice(_DH)
    V = _log(rng, 2000, 157184)
    if kind == "rollout":
        B, Lb = _log(rng, 1, 64), rng.choice([4, 8, 16, 32, 32, 32])
        before, after = rng.randint(0, 7), rng.randint(0, 8)
        prompt = _log(rng, 40, max(64, min(8192, (1 << 29) // (B * Hkv * d))))
        causal = rng.random() < 0.25
        dual = not causal and rng.random() < 0.4
        if rng.random() < 0.4:
            rule = dict(rule="topk", k=rng.choice([1, 2, 2, 4]))
        else:
            rule = dict(rule="threshold", tau=rng.choice([0.8, 0.9, 0.95]))
        return _rollout(B, Hq, Hkv, d, Dh, V, prompt, before, after if dual else 0, Lb, dual=dual, bs=Lb if causal else 0,
                        refresh=rng.random() < 0.7, sampled=rng.random() < 0.25, **rule)
    if kind == "step":
        B = _log(rng, 1, 64)
        prefix = _log(rng, 64, max(64, min(16384, (1 << 29) // (B * Hkv * d))))
        return _step(B, Hq, Hkv, d, Dh, V, prefix, rng.choice([4, 8, 16, 32, 32, 64]), rng.choice([1, 2, 4]), rng.random() < 0.5)
    if kind == "varlen_train":
        return _varlen(_log(rng, 4, 128), Hq, Hkv, d, 1 + rng.randint(0, 63), _log(rng, 64, 600), rng.randint(0, 32), _log(rng, 64, 1024),
                       bs=rng.choice([0, 0, 4, 32]))
    if kind == "diffusion_train":
        L = _log(rng, 256, 4096)
        return _diffusion(_log(rng, 1, max(1, 8 * 4096 // L)), L, Hq, Hkv, d, rng.choice([4, 4, 8, 16, 32]))
    if kind == "logprob":
        return _logprob(_log(rng, 1, 64), _log(rng, 64, 1024), Dh, V, rng.choice([0.15, 0.5, 0.85]))
    bs = rng.choice([4, 4, 8, 32])
    L = _log(rng, 128, 4096) // bs * bs
    return _full(_log(rng, 1, max(1, 32 * 4096 // L)), L, Hq, Hkv, d, Dh, V, bs)


# --------------------------------------------------------------------------------------------------------------------
# what a user has in hand before the call
# --------------------------------------------------------------------------------------------------------------------
class _Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(seed)
        self.host = torch.Generator().manual_seed(seed)

    def normal(self, *shape, std=1.0):
        x = torch.randn(shape, generator=self.g, device=DEV, dtype=BF16)
        return x if std == 1.0 else x.mul_(std)

    def weights(self, V, Dh):
        return self.normal(V, Dh, std=Dh ** -0.25)

    def ints(self, hi, *shape):
        return torch.randint(0, hi, shape, generator=self.g, device=DEV, dtype=I32)

    def host_ints(self, lo, hi, n):
        return torch.randint(lo, hi + 1, (n,), generator=self.host, dtype=I32)

    def order(self, n):
        return torch.randperm(n, generator=self.host)

    def some_masked(self, B, n, m):
        """uint8 [B, n] with m ones a row, at places drawn for each row."""
        order = torch.rand((B, n), generator=self.g, device=DEV).argsort(dim=1).argsort(dim=1)
        return (order < m).to(U8)

    def bernoulli(self, prob, *shape):
        return (torch.rand(shape, generator=self.g, device=DEV) < prob).to(U8)


def _workspace(nbytes):
    return torch.empty(max(16, nbytes), dtype=U8, device=DEV)


def prepare(case, seed):
    r = _Draw(seed)
    return _PREPARE[case["kind"]](case, r, seed)


def _prepare_rollout(c, r, seed):
    n_blocks = c["blocks_before"] + 1 + c["blocks_after"]
    cfg = Config("case", B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], d=c["d"], Dh=c["Dh"], V=c["V"], prompt=c["prompt"], gen=n_blocks * c["Lb"],
                 Lb=c["Lb"], rule=c["rule"], tau=c["tau"], k=c["k"], dual_cache=c["dual"], mask_mode="block_causal" if c["bs"] else "full",
                 bs=c["bs"], refresh=c["refresh"])
    B, Lb, L = cfg.B, cfg.Lb, cfg.L
    g = GpuRollout(cfg, r.weights(cfg.V, cfg.Dh), DEV, sample_seed=seed if c["sampled"] else None, confidence=c["confidence"])
    g.diagnostics = False                     # as a production loop runs it: no extra per-row outputs
    g.x.copy_(r.ints(cfg.V - 1, B, L))
    image = None
    if c["refresh"]:
        image = (r.normal(B, cfg.Hkv, L, cfg.d), r.normal(B, cfg.Hkv, L, cfg.d))
    else:
        g.cache_k.copy_(r.normal(B, cfg.Hkv, L, cfg.d))
        g.cache_v.copy_(r.normal(B, cfg.Hkv, L, cfg.d))
    mask = r.some_masked(B, Lb, c["masked"]) if c["masked"] else None
    # what the model's forward passes bring: fresh queries, block K/V and hidden states for every step a block can take
    steps = [(r.normal(B, Lb, cfg.Hq, cfg.d), r.normal(B, cfg.Hkv, Lb, cfg.d), r.normal(B, cfg.Hkv, Lb, cfg.d), r.normal(B, Lb, cfg.Dh))
             for _ in range(Lb + 1)]
    return dict(kind="rollout", g=g, block=c["blocks_before"], steps=steps, mask=mask, image=image)


def _prepare_step(c, r, seed):
    B, Lb, Hq, Hkv, d, V, P = c["B"], c["Lb"], c["Hq"], c["Hkv"], c["d"], c["V"], c["prefix"]
    n, L = B * Lb, P + Lb
    s = dict(kind="step", case=c, q=r.normal(B, Lb, Hq, d), out=torch.zeros((B, Lb, Hq, d), dtype=BF16, device=DEV),
             cache_k=r.normal(B, Hkv, L, d), cache_v=r.normal(B, Hkv, L, d), kblk=r.normal(B, Hkv, Lb, d), vblk=r.normal(B, Hkv, Lb, d),
             hidden=r.normal(n, c["Dh"]), w=r.weights(V, c["Dh"]), x=r.ints(V - 1, B, L), mask0=r.some_masked(B, Lb, (Lb + 1) // 2))
    s["lens"] = r.host_ints((P + 1) // 2, P, B).to(DEV) if c["ragged"] else None
    s["mask"] = s["mask0"].clone()
    s["rows"] = torch.nonzero(s["mask0"].reshape(-1)).reshape(-1).to(I32)
    for name, dtype in (("conf", F32), ("tok", I32)):
        s[name] = torch.zeros((B, Lb), dtype=dtype, device=DEV)
    s["n_commit"], s["remaining"] = (torch.zeros(B, dtype=I32, device=DEV) for _ in range(2))
    s["next_rows"], s["next_m"] = torch.zeros(n, dtype=I32, device=DEV), torch.zeros(1, dtype=I32, device=DEV)
    s["prefix"] = (s["cache_k"][:, :, :P], s["cache_v"][:, :, :P], 0)
    s["attn_ws"] = _workspace(dlm.block_attn_workspace_bytes(s["q"], prefix=s["prefix"], block=(s["kblk"], s["vblk"], P)))
    s["lm_ws"] = _workspace(dlm.lmhead_workspace_bytes(s["rows"].numel(), V))
    return s


def _prepare_varlen(c, r, seed):
    B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], c["d"]
    # the lengths are the case's own (so that its total is), their order in the batch the seed's
    own = _Draw(sum(c[x] for x in ("prompt_lo", "prompt_hi", "resp_lo", "resp_hi")))
    lens = (own.host_ints(c["prompt_lo"], c["prompt_hi"], B) + own.host_ints(c["resp_lo"], c["resp_hi"], B))[r.order(B)]
    cu = torch.zeros(B + 1, dtype=I32)
    cu[1:] = torch.cumsum(lens, 0)
    T = int(cu[-1])
    s = dict(kind="varlen_train", case=c, cu=cu.to(DEV), longest=int(lens.max()), q=r.normal(T, Hq, d), k=r.normal(T, Hkv, d), v=r.normal(T, Hkv, d),
             d_out=r.normal(T, Hq, d))
    s["out"], s["d_q"], s["d_k"], s["d_v"] = (torch.zeros_like(s[x]) for x in ("q", "q", "k", "k"))
    s["lse"] = torch.zeros((Hq, T), dtype=F32, device=DEV)
    s["ws"] = _workspace(dlm.block_attn_bwd_workspace_bytes(T, Hq))
    return s


def _prepare_diffusion(c, r, seed):
    B, L, Hq, Hkv, d = c["B"], c["L"], c["Hq"], c["Hkv"], c["d"]
    s = dict(kind="diffusion_train", case=c, ws=_workspace(dlm.block_attn_bwd_workspace_bytes(B * L, Hq)))
    for half in ("n", "c"):                   # the noisy and the clean copy
        s["q" + half], s["do" + half] = r.normal(B, L, Hq, d), r.normal(B, L, Hq, d)
        s["k" + half], s["v" + half] = r.normal(B, Hkv, L, d), r.normal(B, Hkv, L, d)
        s["o" + half], s["dq" + half] = torch.zeros_like(s["q" + half]), torch.zeros_like(s["q" + half])
        s["dk" + half], s["dv" + half] = torch.zeros_like(s["k" + half]), torch.zeros_like(s["k" + half])
        s["lse" + half] = torch.zeros((B, Hq, L), dtype=F32, device=DEV)
    # the noisy half's gradient of the clean keys: the caller adds it to the clean half's own
    s["dkx"], s["dvx"] = torch.zeros_like(s["kc"]), torch.zeros_like(s["kc"])
    return s


def _prepare_logprob(c, r, seed):
    B, n, V = c["B"], c["n_pos"], c["V"]
    s = dict(kind="logprob", case=c, hidden=r.normal(B * n, c["Dh"]), w=r.weights(V, c["Dh"]), target=r.ints(V - 1, B * n),
             mask=r.bernoulli(c["mask_prob"], B, n))
    s["mask"][:, 0] = 1                       # at least one term a sequence
    s["weight"] = torch.full((B,), -1.0 / c["mask_prob"], dtype=F32, device=DEV)
    s["rows"] = torch.nonzero(s["mask"].reshape(-1)).reshape(-1).to(I32)
    for name, dtype in (("conf", F32), ("tok", I32), ("lse", F32), ("zt", F32)):
        s[name] = torch.zeros(B * n, dtype=dtype, device=DEV)
    s["out"], s["terms"] = torch.zeros(B, dtype=F32, device=DEV), torch.zeros(B, dtype=I32, device=DEV)
    s["ws"] = _workspace(dlm.lmhead_workspace_bytes(s["rows"].numel(), V))
    return s


def _prepare_full(c, r, seed):
    B, L, Hq, Hkv, d, V = c["B"], c["L"], c["Hq"], c["Hkv"], c["d"], c["V"]
    n = B * L
    s = dict(kind="full_pass", case=c, q=r.normal(B, L, Hq, d), k=r.normal(B, Hkv, L, d), v=r.normal(B, Hkv, L, d), hidden=r.normal(n, c["Dh"]),
             w=r.weights(V, c["Dh"]), x=r.ints(V - 1, B, L), mask0=r.bernoulli(0.5, B, L))
    s["mask"] = s["mask0"].clone()
    s["out"] = torch.zeros_like(s["q"])
    s["lse"] = torch.zeros((B, Hq, L), dtype=F32, device=DEV)
    s["conf"], s["tok"] = torch.zeros((B, L), dtype=F32, device=DEV), torch.zeros((B, L), dtype=I32, device=DEV)
    s["n_commit"], s["remaining"] = (torch.zeros(B, dtype=I32, device=DEV) for _ in range(2))
    s["rows"], s["m"] = torch.zeros(n, dtype=I32, device=DEV), torch.zeros(1, dtype=I32, device=DEV)
    s["next_rows"], s["next_m"] = torch.zeros(n, dtype=I32, device=DEV), torch.zeros(1, dtype=I32, device=DEV)
    s["n_masked"] = int(s["mask0"].sum())     # the caller drew the mask and knows how many positions it hid
    s["lm_ws"] = _workspace(dlm.lmhead_workspace_bytes(s["n_masked"], V))
    return s


_PREPARE = dict(rollout=_prepare_rollout, step=_prepare_step, varlen_train=_prepare_varlen, diffusion_train=_prepare_diffusion,
                logprob=_prepare_logprob, full_pass=_prepare_full)


# --------------------------------------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------------------------------------
def run(state):
    return _RUN[state["kind"]](state)


def _run_rollout(s):
    g = s["g"]
    steps = s["steps"]
    g.run_block(s["block"], lambda block, step: steps[step], init_mask=s["mask"], refresh=s["image"])
    return dict(x=g.x, mask=g.mask, cache_k=g.cache_k, cache_v=g.cache_v, out=g.O, conf=g.conf, tok=g.tok, commit_now=g.commit_now)


def _run_step(s):
    c = s["case"]
    s["mask"].copy_(s["mask0"])               # the block's state before this step
    dlm.block_attn(s["q"], s["out"], prefix=s["prefix"], block=(s["kblk"], s["vblk"], c["prefix"]), prefix_len_b=s["lens"], workspace=s["attn_ws"])
    dlm.lmhead_confidence(s["hidden"], s["w"], s["conf"], s["tok"], row_idx=s["rows"], forbid_token=c["V"] - 1, out_scatter=True, workspace=s["lm_ws"])
    dlm.unmask_commit(s["conf"], s["tok"], s["x"], s["mask"], s["n_commit"], s["remaining"], x_pos0=c["prefix"], rule=dlm.RULE_TOPK, k=c["k"],
                      next_row_idx=s["next_rows"], next_m=s["next_m"])
    # (the row list's tail past its length is not defined by the call and does not change here)
    return dict(out=s["out"], conf=s["conf"], tok=s["tok"], x=s["x"], mask=s["mask"], n_commit=s["n_commit"], remaining=s["remaining"],
                next_rows=s["next_rows"], next_m=s["next_m"])


def _run_varlen(s):
    c = s["case"]
    mask = dict(mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=c["bs"]) if c["bs"] else {}
    dlm.varlen_attn(s["q"], s["k"], s["v"], s["out"], s["cu"], s["longest"], lse=s["lse"], **mask)
    dlm.block_attn_bwd(s["q"], s["out"], s["d_out"], s["lse"], s["d_q"], block=(s["k"], s["v"]), d_block=(s["d_k"], s["d_v"]), cu_seqlens=s["cu"],
                       max_seqlen=s["longest"], workspace=s["ws"], **mask)
    return {x: s[x] for x in ("out", "lse", "d_q", "d_k", "d_v")}


def _run_diffusion(s):
    mask = dict(mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=s["case"]["bs"])
    clean, noisy = (s["kc"], s["vc"], 0, dlm.SEG_EARLIER_BLOCKS), (s["kn"], s["vn"], 0, dlm.SEG_SAME_BLOCK)
    own = (s["kc"], s["vc"], 0)
    dlm.block_attn(s["qn"], s["on"], prefix=clean, block=noisy, lse=s["lsen"], **mask)
    dlm.block_attn(s["qc"], s["oc"], block=own, lse=s["lsec"], **mask)
    dlm.block_attn_bwd(s["qn"], s["on"], s["don"], s["lsen"], s["dqn"], prefix=clean, block=noisy, d_prefix=(s["dkx"], s["dvx"]),
                       d_block=(s["dkn"], s["dvn"]), workspace=s["ws"], **mask)
    dlm.block_attn_bwd(s["qc"], s["oc"], s["doc"], s["lsec"], s["dqc"], block=own, d_block=(s["dkc"], s["dvc"]), workspace=s["ws"], **mask)
    return {x: s[x] for x in ("on", "lsen", "oc", "lsec", "dqn", "dkn", "dvn", "dkx", "dvx", "dqc", "dkc", "dvc")}


def _run_logprob(s):
    dlm.lmhead_confidence(s["hidden"], s["w"], s["conf"], s["tok"], row_idx=s["rows"], forbid_token=s["case"]["V"] - 1, out_scatter=True, lse=s["lse"],
                          target=s["target"], ztarget=s["zt"], workspace=s["ws"])
    dlm.seq_logprob(s["zt"], s["lse"], s["mask"], s["out"], weight=s["weight"], n_terms=s["terms"])
    return {x: s[x] for x in ("conf", "tok", "lse", "zt", "out", "terms")}


def _run_full(s):
    c = s["case"]
    s["mask"].copy_(s["mask0"])
    dlm.block_attn(s["q"], s["out"], block=(s["k"], s["v"], 0), mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=c["bs"], lse=s["lse"])
    dlm.mask_compact(s["mask"], s["rows"], s["m"])
    dlm.lmhead_confidence(s["hidden"], s["w"], s["conf"], s["tok"], M=s["n_masked"], row_idx=s["rows"], m_dev=s["m"], forbid_token=c["V"] - 1,
                          out_scatter=True, workspace=s["lm_ws"])
    dlm.unmask_commit(s["conf"], s["tok"], s["x"], s["mask"], s["n_commit"], s["remaining"], x_pos0=0, group_len=c["bs"], rule=dlm.RULE_THRESHOLD,
                      threshold=0.95, next_row_idx=s["next_rows"], next_m=s["next_m"])
    return {x: s[x] for x in ("out", "lse", "conf", "tok", "x", "mask", "n_commit", "remaining", "next_m")}


_RUN = dict(rollout=_run_rollout, step=_run_step, varlen_train=_run_varlen, diffusion_train=_run_diffusion, logprob=_run_logprob, full_pass=_run_full)


# --------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------------------------------------
def _confident(Dh, V, tau):
    """Share of positions whose arg-max probability reaches tau: logits are N(0, Dh^1/2), whose largest few of V form a Poisson process of
    exponential intensity with scale s = Dh^1/4 / sqrt(2 ln V); the normalised weights then follow the Poisson-Dirichlet law of index 1 / s."""
    a = math.sqrt(2 * math.log(V)) / Dh ** 0.25
    if a >= 1:
        return 0.0
    return (1 - tau) ** a / a * math.sin(math.pi * a) / math.pi


def _masked_per_step(c):
    """Expected positions per sequence that are still masked before each step of a block."""
    m, got = float(c["masked"] or c["Lb"]), []
    share = 0.0 if c["rule"] == "topk" else _confident(c["Dh"], c["V"], c["tau"])
    while m > 0.5 and len(got) <= c["Lb"]:
        got.append(m)
        m -= c["k"] if c["rule"] == "topk" else max(min(1.0, m), share * m)
    return got


def _lmhead_work(rows, Dh, V):
    return 2.0 * V * Dh + 2.0 * rows * Dh + 8.0 * rows, 2.0 * rows * Dh * V


def work(case):
    c, kind = case, case["kind"]
    if kind == "rollout":
        P, S = c["prompt"] + c["blocks_before"] * c["Lb"], c["blocks_after"] * c["Lb"] if c["dual"] else 0
        keys, rows_q = P + S + c["Lb"], c["Lb"] * c["Hq"]
        nbytes = 8.0 * c["B"] * c["Hkv"] * (P + S) * c["d"] if c["refresh"] else 0.0
        nbytes += 8.0 * c["B"] * c["Hkv"] * c["Lb"] * c["d"]          # the finished block's K/V into the cache
        flops = 0.0
        for m in _masked_per_step(c):
            lb, lf = _lmhead_work(m * c["B"], c["Dh"], c["V"])
            nbytes += c["B"] * c["d"] * (4.0 * c["Hkv"] * keys + 4.0 * rows_q) + lb
            flops += 4.0 * c["B"] * c["d"] * rows_q * keys + lf
        return dict(bytes=nbytes, flops=flops)
    if kind == "step":
        keys = c["prefix"] * (0.75 if c["ragged"] else 1.0) + c["Lb"]
        lb, lf = _lmhead_work(c["B"] * ((c["Lb"] + 1) // 2), c["Dh"], c["V"])
        rows_q = c["Lb"] * c["Hq"]
        return dict(bytes=c["B"] * c["d"] * (4.0 * c["Hkv"] * keys + 4.0 * rows_q) + lb, flops=4.0 * c["B"] * c["d"] * rows_q * keys + lf)
    if kind == "varlen_train":
        # lengths are sums of two uniform draws: mean and mean square in closed form
        mean = (c["prompt_lo"] + c["prompt_hi"] + c["resp_lo"] + c["resp_hi"]) / 2.0
        square = mean * mean + ((c["prompt_hi"] - c["prompt_lo"]) ** 2 + (c["resp_hi"] - c["resp_lo"]) ** 2) / 12.0
        pairs = c["B"] * (square if not c["bs"] else (square + mean * c["bs"]) / 2)
        tokens = c["B"] * mean
        # forward: Q, K, V in, O out; backward: Q, K, V, O, dO in, dQ, dK, dV out
        return dict(bytes=2.0 * tokens * c["d"] * (6 * c["Hq"] + 6 * c["Hkv"]), flops=14.0 * c["Hq"] * c["d"] * pairs)
    if kind == "diffusion_train":
        pairs = c["B"] * c["L"] * ((c["L"] + c["bs"]) / 2.0)            # of each half: every earlier block and the own one
        return dict(bytes=2.0 * c["B"] * c["L"] * c["d"] * (12 * c["Hq"] + 16 * c["Hkv"]), flops=2 * 14.0 * c["Hq"] * c["d"] * pairs)
    if kind == "logprob":
        rows = c["B"] * c["n_pos"] * c["mask_prob"]
        lb, lf = _lmhead_work(rows, c["Dh"], c["V"])
        return dict(bytes=lb + 12.0 * rows, flops=lf)
    rows = c["B"] * c["L"] * 0.5
    lb, lf = _lmhead_work(rows, c["Dh"], c["V"])
    pairs = c["B"] * c["L"] * ((c["L"] + c["bs"]) / 2.0)
    return dict(bytes=lb + 4.0 * c["B"] * c["L"] * c["d"] * (c["Hq"] + c["Hkv"]) + 14.0 * c["B"] * c["L"],
                flops=lf + 4.0 * c["Hq"] * c["d"] * pairs)


def tolerance(case):
    # LM head: 32-bit sums over Dh; against 64-bit logits the confidences are off by 4.3e-6 (2-norm) and the log-sum-exps by 2.7e-7, another
    # order of summation by 5.1e-6; a token differs only at a tie.
    # Attention: probabilities and results rounded to bf16; outputs are off by 2.1e-3 to 2.3e-3 against 64-bit, gradients by 2.3e-3 to 2.7e-3,
    # and by 3.0e-3 to 3.1e-3 against the same path with its sums split another way.
    if case["kind"] == "logprob":
        return dict(rel=2e-5, differ=1e-3)
    return dict(rel=1.2e-2, differ=5e-3)
