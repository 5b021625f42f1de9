"""Every shape of the backward kernels at the sizes where it can go wrong: keys and rows around a wavefront's 64 and a workgroup's
128, group sizes that do and do not divide a 32-row tile, token strides that do not fit 32-bit offsets.  The batch decides which
shape runs: 1 sequence with 256 rows a KV head and more takes the row-split dK / dV kernel, fewer rows or more than 256 slabs of 128
keys the key-split one, with at most 64 keys one wavefront a workgroup of it; 1024 workgroups of 128 rows and more with 256 keys and
more (384 under a block-causal mask), d = 128, the 64-row dQ kernel.  All sequences of a batch are copies of one, so the first is
checked against the oracle and the others have to have its bits."""
import numpy as np
import pytest
import torch

from oracle import KV
from oracle import backward as obw
from paper_2604_04215_amd import binding as dlm
from paper_2604_04215_amd import synth
from gpu_util import DEV, GuardedWorkspace, bf16_dev, bf16_host, dev, rnd
from test_gpu_attn_bwd import FRO_TOL, fro_err, make, run_bwd

pytestmark = pytest.mark.gpu


def batches(L, Hq, Hkv):
    slabs, rows = (L + 127) // 128 * Hkv, (L * (Hq // Hkv) + 127) // 128 * Hkv
    return [1, 256 // slabs + 1, (1024 + rows - 1) // rows]


def error_bounds(q, segs, d_out, mode="full", bs=0, q_pos0=0):
    """Per element of (dQ, dK and dV of each segment): 6 standard deviations of the error that the roundings to bf16 leave (8 significant
    bits: independent, uniform within 2^-8 of the value or less, so of deviation u = 2^-8 / sqrt 3 or less), to first order:
      forward   O: the probabilities of its product and the result, u^2 (sum_j P^2 V^2 + O^2), so for delta = sum_c dO O
                the sum of that times dO^2
      backward  dV: P in the product; dK, dQ: dS in the product, and delta, which shifts all dS of a row by P times its error; the results
    The 32-bit sums, exponentials and log-sum-exps are off by some 1e-6 and do not show.  The largest error seen is 0.6 of this."""
    u = 2.0 ** -8 / 3 ** 0.5
    (B, Lq, Hq, d), f64 = q.shape, synth.bf16_bits_to_f64
    segs = [x for x in segs if x is not None]
    k, v = (np.concatenate([f64(x.k if what == "k" else x.v) for x in segs], axis=2)[0] for what in "kv")
    g, scale, vis = Hq // k.shape[0], d ** -0.5, obw.visibility(Lq, segs, mask_mode=mode, bs=bs, q_pos0=q_pos0)
    e_q, e_k, e_v = np.zeros((Lq, Hq, d)), np.zeros(k.shape), np.zeros(k.shape)
    grad_k, grad_v = np.zeros(k.shape), np.zeros(k.shape)
    for h in range(Hq):
        kh, Q, dO = h // g, f64(q)[0, :, h], f64(d_out)[0, :, h]
        K, V = k[kh], v[kh]
        s = np.where(vis, scale * (Q @ K.T), -np.inf)
        P = np.exp(s - np.where(vis.any(1), s.max(1), 0)[:, None])
        P /= np.where(vis.any(1), P.sum(1), 1)[:, None]
        dP, O = dO @ V.T, P @ V
        dS = P * (dP - (P * dP).sum(1, keepdims=True))
        delta = (dO ** 2 * u ** 2 * (P ** 2 @ V ** 2 + O ** 2)).sum(1)
        dQ = scale * (dS @ K)
        e_q[:, h] = scale ** 2 * (u ** 2 * (dS ** 2 @ K ** 2) + (P @ K) ** 2 * delta[:, None]) + u ** 2 * dQ ** 2
        e_k[kh] += scale ** 2 * ((u ** 2 * dS ** 2 + P ** 2 * delta[:, None]).T @ Q ** 2)
        e_v[kh] += u ** 2 * (P ** 2).T @ dO ** 2
        grad_k[kh] += scale * dS.T @ Q
        grad_v[kh] += P.T @ dO
    e_k, e_v = e_k + u ** 2 * grad_k ** 2, e_v + u ** 2 * grad_v ** 2
    ends = np.cumsum([0] + [x.len for x in segs])
    cut = lambda e: [6 * np.sqrt(e[None, :, a:z]) for a, z in zip(ends, ends[1:])]
    return [6 * np.sqrt(e_q[None])] + [e for pair in zip(cut(e_k), cut(e_v)) for e in pair]


def assert_close(got_u16, ref, bound):
    """The largest difference over its bound, and in aggregate: a wrong or missing term of many elements shows there first."""
    diff = np.abs(synth.bf16_bits_to_f64(got_u16).reshape(ref.shape) - ref)
    worst = float((diff / np.maximum(bound, 1e-7)).max())
    assert worst <= 1.0 and fro_err(got_u16, ref) <= FRO_TOL, (worst, fro_err(got_u16, ref))


def check_copies(q, segs, d_out, B, **mask):
    rep = lambda x: np.repeat(x, B, axis=0)
    dq, grads = run_bwd(rep(q), [None if s is None else KV(rep(s.k), rep(s.v), s.pos0, s.rule) for s in segs], rep(d_out), **mask)
    rdq, rg = obw.attention_backward(q, [s for s in segs if s is not None], d_out, mask_mode=mask.get("mode", "full"),
                                     **{x: mask[x] for x in mask if x != "mode"})
    pairs = [(dq, rdq)] + [(got, ref) for g, r in zip([g for g in grads if g is not None], rg) for got, ref in zip(g, r)]
    for (got, ref), bound in zip(pairs, error_bounds(q, segs, d_out, **mask)):
        assert (got == got[:1]).all()
        assert_close(got[:1], ref, bound)


@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
@pytest.mark.parametrize("L,Hq,Hkv,d,bs", [(63, 2, 2, 128, 0), (65, 7, 1, 64, 0), (127, 8, 1, 128, 4), (129, 3, 1, 128, 32), (257, 4, 1, 64, 8),
                                           (260, 7, 1, 128, 4), (31, 64, 1, 64, 0), (1, 1, 1, 128, 1)])
def test_edges(size, L, Hq, Hkv, d, bs):
    q, segs, d_out = make(1, L, Hq, Hkv, d, (0, L, 0), seed=3000 + L)
    check_copies(q, segs, d_out, batches(L, Hq, Hkv)[size], **(dict(mode="block_causal", bs=bs) if bs else {}))


@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
def test_segments(size):
    q, segs, d_out = make(1, 132, 4, 2, 128, (132, 132, 0), seed=3400, pos=(0, 0, 0), rules=("earlier", "same", "causal"))
    check_copies(q, segs, d_out, batches(132, 4, 2)[size], mode="block_causal", bs=4)
    q, segs, d_out = make(1, 40, 8, 2, 128, (33, 40, 70), seed=3500)
    check_copies(q, segs, d_out, batches(40, 8, 2)[size])


@pytest.mark.parametrize("L,Hq,Hkv,bs", [(255, 1, 1, 0), (256, 2, 1, 0), (257, 1, 1, 0), (319, 3, 1, 0), (383, 7, 1, 4), (384, 2, 2, 32),
                                         (415, 7, 1, 4), (450, 3, 1, 32)])
def test_dq64_edges(L, Hq, Hkv, bs):
    q, segs, d_out = make(1, L, Hq, Hkv, 128, (0, L, 0), seed=3250 + L)
    check_copies(q, segs, d_out, batches(L, Hq, Hkv)[2], **(dict(mode="block_causal", bs=bs) if bs else {}))


@pytest.mark.parametrize("lens,mask", [
    ((150, 40, 70), {}), ((0, 40, 230), {}), ((300, 0, 0), {}), ((31, 40, 200), {}),
    ((400, 40, 0), dict(mode="block_causal", bs=16, q_pos0=400)), ((385, 40, 64), dict(mode="block_causal", bs=7, q_pos0=385))])
def test_dq64_segments(lens, mask):
    q, segs, d_out = make(1, 40, 8, 2, 128, lens, seed=3260 + lens[0])
    check_copies(q, segs, d_out, batches(40, 8, 2)[2], **mask)


def test_dq64_block_diffusion():
    q, segs, d_out = make(1, 388, 4, 2, 128, (388, 388, 0), seed=3270, pos=(0, 0, 0), rules=("earlier", "same", "causal"))
    check_copies(q, segs, d_out, batches(388, 4, 2)[2], mode="block_causal", bs=4)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,Hq,Hkv,bs", [(1, 1, 1, 0), (31, 2, 2, 0), (33, 3, 1, 4), (63, 8, 1, 0), (64, 7, 1, 32), (64, 1, 1, 4), (65, 2, 1, 0)])
def test_at_most_64_keys(d, L, Hq, Hkv, bs):
    """513 (sequence, KV head) pairs and more: one wavefront a workgroup up to 64 keys; 1 to 16 tiles of 32 rows."""
    q, segs, d_out = make(1, L, Hq, Hkv, d, (0, L, 0), seed=3300 + L)
    check_copies(q, segs, d_out, 513 // Hkv + 1, **(dict(mode="block_causal", bs=bs) if bs else {}))


@pytest.mark.parametrize("d", [64, 128])
def test_at_most_64_keys_a_segment(d):
    q, segs, d_out = make(1, 60, 4, 1, d, (60, 60, 0), seed=3310, pos=(0, 0, 0), rules=("earlier", "same", "causal"))
    check_copies(q, segs, d_out, 520, mode="block_causal", bs=4)
    q, segs, d_out = make(1, 40, 4, 1, d, (33, 40, 70), seed=3320)
    check_copies(q, segs, d_out, 520)


@pytest.mark.parametrize("L,Hq,Hkv", [(256, 1, 1), (255, 1, 1), (86, 6, 2), (85, 6, 2)])
@pytest.mark.parametrize("d,bs", [(64, 0), (64, 4), (128, 0), (128, 32)])
def test_around_the_fewest_rows_of_a_row_split(L, Hq, Hkv, d, bs):
    """256 rows a KV head and the next fewer, with few, 128 and 129 slabs of 128 keys (where 512 rows would be needed)."""
    for B in (1, 128 // ((L + 127) // 128 * Hkv), 128 // ((L + 127) // 128 * Hkv) + 1):
        q, segs, d_out = make(1, L, Hq, Hkv, d, (0, L, 0), seed=3550 + L)
        check_copies(q, segs, d_out, B, **(dict(mode="block_causal", bs=bs) if bs else {}))


@pytest.mark.parametrize("B", [16, 32], ids=["row-split", "key-split"])
def test_paired_slabs(B):
    """33 slabs of 64 keys (17 of 128), 1024 of them and more: the launch of two wavefronts side by side (32 sequences) pairs the slabs of a block-causal
    segment; the row-split one (16) has as many and does not."""
    q, segs, d_out = make(1, 2100, 2, 2, 64, (0, 2100, 0), seed=3600)
    check_copies(q, segs, d_out, B, mode="block_causal", bs=32)


@pytest.mark.parametrize("L,g,bs,rules", [(388, 4, 4, None), (520, 7, 8, None), (642, 4, 32, None), (388, 4, 4, ("earlier", "same", "causal")),
                                          (516, 7, 4, ("earlier", "same", "causal"))])
def test_paired_slabs_at_128(L, g, bs, rules):
    """4, 5 and 6 slabs of 128 keys (odd: the middle one has no partner), 1024 of them and more; the grouped 1-D grid and the plain one
    give the same bits."""
    q, segs, d_out = make(1, L, g, 1, 128, (L, L, 0) if rules else (0, L, 0), seed=3650 + L, **(dict(pos=(0, 0, 0), rules=rules) if rules else {}))
    B = 1024 // ((L + 127) // 128) + 1
    check_copies(q, segs, d_out, B, mode="block_causal", bs=bs)
    rep = lambda x: np.repeat(x, B, axis=0)
    res = []
    try:
        for remap in (7, 0):
            dlm.set_option("attn_remap", remap)
            res.append(run_bwd(rep(q), [None if x is None else KV(rep(x.k), rep(x.v), x.pos0, x.rule) for x in segs], rep(d_out), mode="block_causal", bs=bs))
    finally:
        dlm.set_option("attn_remap", 7)
    for (x, y) in zip(res[0][1], res[1][1]):
        assert x is y is None or all(np.array_equal(a, r) for a, r in zip(x, y))
    assert np.array_equal(res[0][0], res[1][0])


@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
@pytest.mark.parametrize("d", [64, 128])
def test_rows_that_see_no_key(size, d):
    """The earlier blocks alone: the first block's rows see nothing."""
    q, segs, d_out = make(1, 388, 4, 1, d, (388, 0, 0), seed=3690, pos=(0, 0, 0), rules=("earlier", "same", "causal"))
    check_copies(q, segs, d_out, batches(388, 4, 1)[size], mode="block_causal", bs=4)


@pytest.mark.parametrize("size", [0, 1], ids=["row-split", "key-split"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,Hq,Hkv,lens,bs", [(64, 5, 1, None, 0), (96, 3, 1, None, 4), (255, 14, 2, None, 32), (257, 7, 1, None, 0), (320, 6, 2, None, 7),
                                              (96, 7, 1, (70, 96, 40), 0), (256, 7, 1, (256, 256, 0), 4)])
def test_heads_apart(size, d, L, Hq, Hkv, lens, bs):
    """Heads that do not divide a 32-row tile and rows that fill theirs: dK / dV takes the heads one after another (257 rows: too many tiles for it; d = 128 with
    a causal mask: the kernel without that walk, on the same rows), with as few as one tile a head for four wavefronts (late keys of a causal mask) and an
    own-block segment's range in the middle."""
    rules = ("earlier", "same", "causal") if lens and bs else None
    q, segs, d_out = make(1, L, Hq, Hkv, d, lens or (0, L, 0), seed=3800 + L, **(dict(pos=(0, 0, 0), rules=rules) if rules else {}))
    check_copies(q, segs, d_out, batches(L, Hq, Hkv)[size], **(dict(mode="block_causal", bs=bs) if bs else {}))


@pytest.mark.parametrize("L,Hq,Hkv,bs,rules", [(512, 7, 1, 4, None), (640, 7, 1, 32, None), (639, 6, 2, 8, None), (512, 7, 1, 4, ("earlier", "same", "causal"))])
def test_heads_apart_on_paired_slabs(L, Hq, Hkv, bs, rules):
    """4 and 5 slabs of 128 keys, 1024 of them and more, of heads of 64 that do not divide a tile: the second slab of a pair is walked upwards, head after
    head, from where its causal range begins (an odd number of slabs: the middle one has no partner)."""
    q, segs, d_out = make(1, L, Hq, Hkv, 64, (L, L, 0) if rules else (0, L, 0), seed=3850 + L, **(dict(pos=(0, 0, 0), rules=rules) if rules else {}))
    check_copies(q, segs, d_out, 1024 // ((L + 127) // 128 * Hkv) + 1, mode="block_causal", bs=bs)


class Backwards:
    """The tokens of x [B, L, H, d] as the binding sees a tensor, last one first in memory: a negative token stride."""
    def __init__(self, x):
        self.flipped = x.flip(1).contiguous()
        self.shape, self.dtype, self.is_cuda = x.shape, x.dtype, x.is_cuda
        self.dim, self.numel = x.dim, x.numel

    def stride(self, i):
        st = self.flipped.stride(i)
        return -st if i == 1 else st

    def data_ptr(self):
        return self.flipped[:, -1].data_ptr()


@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
@pytest.mark.parametrize("layout", ["heads first", "heads first, backwards", "backwards"])
@pytest.mark.parametrize("g,d,bs", [(4, 128, 0), (7, 128, 4), (4, 64, 4), (7, 64, 0)])
def test_layouts(size, layout, g, d, bs):
    """Q and dO laid out differently (with 4 heads a group a tile still holds whole queries) and tokens backwards in memory."""
    L = 386
    B = batches(L, g, 1)[size]
    mask = dict(mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=bs) if bs else {}
    q, segs, d_out = make(1, L, g, 1, d, (0, L, 0), seed=3720 + L)
    rep = lambda x: bf16_dev(np.repeat(x, B, axis=0))
    qd, kd, vd, dod = rep(q), rep(segs[1].k), rep(segs[1].v), rep(d_out)
    out, dk, dv = (torch.empty_like(x) for x in (qd, kd, vd))
    lse = torch.empty((B, g, L), dtype=torch.float32, device=DEV)
    dlm.block_attn(qd, out, block=(kd, vd, 0), lse=lse, **mask)
    dq = torch.empty_like(qd)
    if "heads first" in layout:
        dod = dod.transpose(1, 2).contiguous().transpose(1, 2)
    if "backwards" in layout:
        qd, out = Backwards(qd), Backwards(out)
        dod = dod if "heads first" in layout else Backwards(dod)
    ws = torch.empty(dlm.block_attn_bwd_workspace_bytes(B * L, g), dtype=torch.uint8, device=DEV)
    dlm.block_attn_bwd(qd, out, dod, lse, dq, block=(kd, vd, 0), d_block=(dk, dv), workspace=ws, **mask)
    oracle_mask = dict(mode="block_causal", bs=bs) if bs else {}
    rq, [(rk, rv)] = obw.attention_backward(q, [segs[1]], d_out, mask_mode=oracle_mask.get("mode", "full"), bs=bs)
    for got, ref, bound in zip((dq, dk, dv), (rq, rk, rv), error_bounds(q, segs, d_out, **oracle_mask)):
        h = bf16_host(got)
        assert (h == h[:1]).all()
        assert_close(h[:1], ref, bound)


PACKED = (400, 1, 65, 0, 129, 63, 257, 33)


@pytest.mark.parametrize("groups", [10, 19], ids=["single", "paired"])
@pytest.mark.parametrize("g,bs,d", [(2, 0, 128), (7, 0, 128), (2, 4, 128), (7, 32, 128), (7, 32, 64), (3, 4, 64)])
def test_packed(groups, g, bs, d):
    """Unequal sequences, many enough for the 64-row dQ and the key-split dK / dV kernels (80 of them: 1120 workgroups of 128 rows, 640
    slabs) and, under the block-causal mask, for paired slabs (152: 1216).  The lengths come in groups of 8, the same 8
    sequences each time and in another order.  At d = 64 7 and 3 heads are taken one after another in the sequences whose tiles they fill."""
    Hkv = 2
    Hq = g * Hkv
    starts = np.concatenate([[0], np.cumsum(PACKED)])
    n = int(starts[-1])
    q, k, v, d_out = rnd(41, (n, Hq, d)), rnd(42, (n, Hkv, d)), rnd(43, (n, Hkv, d)), rnd(44, (n, Hq, d))
    which = np.concatenate([np.roll(np.arange(8), i) for i in range(groups)])
    lens = np.array(PACKED)[which]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    take = np.concatenate([np.arange(starts[s], starts[s + 1]) for s in which])
    qd, kd, vd, dod = (bf16_dev(x[take]) for x in (q, k, v, d_out))
    T = len(take)
    mask = dict(mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=bs) if bs else {}
    out, (dq, dk, dv) = torch.empty_like(qd), (torch.full_like(x, float("nan")) for x in (qd, kd, vd))
    lse = torch.empty((Hq, T), dtype=torch.float32, device=DEV)
    dlm.varlen_attn(qd, kd, vd, out, dev(cu), max(PACKED), lse=lse, **mask)
    gw = GuardedWorkspace(dlm.block_attn_bwd_workspace_bytes(T, Hq))
    dlm.block_attn_bwd(qd, out, dod, lse, dq, block=(kd, vd), d_block=(dk, dv), cu_seqlens=dev(cu), max_seqlen=max(PACKED), workspace=gw.ws, **mask)
    gw.check()
    got = [bf16_host(x) for x in (dq, dk, dv)]
    oracle_mask = dict(mode="block_causal", bs=bs) if bs else {}
    heads_first = lambda x: np.ascontiguousarray(x.transpose(1, 0, 2))[None]
    for s in range(8):
        if PACKED[s] == 0:
            continue
        own = slice(starts[s], starts[s + 1])
        q1, seg, do1 = q[own][None], KV(heads_first(k[own]), heads_first(v[own]), 0), d_out[own][None]
        rq, [(rk, rv)] = obw.attention_backward(q1, [seg], do1, mask_mode=oracle_mask.get("mode", "full"), bs=bs)
        bounds = error_bounds(q1, [seg], do1, **oracle_mask)
        at = [i for i in range(len(which)) if which[i] == s]
        for x, ref, bound, kv in zip(got, (rq, rk, rv), bounds, (False, True, True)):
            first = x[cu[at[0]]:cu[at[0] + 1]]
            assert all(np.array_equal(x[cu[i]:cu[i + 1]], first) for i in at)
            assert_close(heads_first(first) if kv else first[None], ref, bound)


@pytest.mark.parametrize("what", ["q", "kv"])
@pytest.mark.parametrize("size,Hq,P", [(0, 7, 0), (0, 3, 0), (1, 3, 0), (2, 3, 0), (2, 3, 256)], ids=["row-split", "key-split-1", "key-split", "dq32", "dq64"])
def test_strides_beyond_32_bit_offsets(size, Hq, P, what):
    """Token strides of 2^23 elements (2^24 bytes) and more leave the 32-bit offsets of the tile requests (a prefix of P keys has
    none of them: it only makes enough keys)."""
    L, Hkv, d, st = 40, 1, 128, (1 << 23) + 8
    B = batches(L, Hq, Hkv)[size]
    q, segs, d_out = make(1, L, Hq, Hkv, d, (P, L, 0), seed=3700)
    prefix = tuple(bf16_dev(np.repeat(x, B, axis=0)) for x in (segs[0].k, segs[0].v)) + (0,) if P else None

    def spread(x):        # [1, L, H, d] -> B copies with token stride st, side by side inside it
        H = x.shape[2]
        t = torch.zeros(L * st, dtype=torch.bfloat16, device=DEV).as_strided((B, L, H, d), (H * d, st, d, 1))
        return t.copy_(x.expand(B, L, H, d))
    wide = spread if what == "q" else lambda x: x.expand(B, *x.shape[1:]).contiguous()
    wide_kv = (lambda x: spread(x.transpose(1, 2)).transpose(1, 2)) if what == "kv" else lambda x: x.expand(B, *x.shape[1:]).contiguous()
    qd, dod = wide(bf16_dev(q)), wide(bf16_dev(d_out))
    kd, vd, dk, dv = (wide_kv(bf16_dev(x)) for x in (segs[1].k, segs[1].v, segs[1].k, segs[1].v))
    out = torch.empty((B, L, Hq, d), dtype=torch.bfloat16, device=DEV)
    lse = torch.empty((B, Hq, L), dtype=torch.float32, device=DEV)
    dlm.block_attn(qd, out, prefix=prefix, block=(kd, vd, P), lse=lse)
    dq = torch.empty_like(out)
    ws = torch.empty(dlm.block_attn_bwd_workspace_bytes(B * L, Hq), dtype=torch.uint8, device=DEV)
    dlm.block_attn_bwd(qd, out, dod, lse, dq, prefix=prefix, block=(kd, vd, P), d_block=(dk, dv), workspace=ws)
    rq, grads = obw.attention_backward(q, segs, d_out)
    bounds = error_bounds(q, segs, d_out)
    for got, ref, bound in zip((dq, dk, dv), (rq, *grads[-1]), (bounds[0], *bounds[-2:])):
        h = bf16_host(got.contiguous())
        assert (h == h[:1]).all()
        assert_close(h[:1], ref, bound)


def test_millions_of_heads_a_group():
    """7 715 248 query heads on one KV head: the place of a row inside its group needs more than the 24 bits of an fp32 quotient.  Only
    heads at a group's two ends have an upstream gradient, so the oracle needs those alone; the last tile of a query's heads runs into the
    next query's."""
    g, L, d = 7715248, 2, 64
    q, segs, d_out = make(1, L, 4, 1, d, (0, L, 0), seed=3800)
    heads = torch.tensor([0, 1, g - 2, g - 1], device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(3800)
    qd = torch.randn((1, L, g, d), generator=gen, device=DEV, dtype=torch.bfloat16)
    dod = torch.zeros_like(qd)
    qd[:, :, heads], dod[:, :, heads] = bf16_dev(q), bf16_dev(d_out)
    kd, vd = bf16_dev(segs[1].k), bf16_dev(segs[1].v)
    out, dq, dk, dv = (torch.empty_like(x) for x in (qd, qd, kd, vd))
    lse = torch.empty((1, g, L), dtype=torch.float32, device=DEV)
    dlm.block_attn(qd, out, block=(kd, vd, 0), lse=lse)
    ws = torch.empty(dlm.block_attn_bwd_workspace_bytes(L, g), dtype=torch.uint8, device=DEV)
    dlm.block_attn_bwd(qd, out, dod, lse, dq, block=(kd, vd, 0), d_block=(dk, dv), workspace=ws)
    rq, [(rk, rv)] = obw.attention_backward(q, [segs[1]], d_out)
    assert int(torch.count_nonzero(dq)) == int(torch.count_nonzero(dq[:, :, heads]))
    for got, ref, bound in zip((dq[:, :, heads], dk, dv), (rq, rk, rv), error_bounds(q, [segs[1]], d_out)):
        assert_close(bf16_host(got), ref, bound)


@pytest.mark.parametrize("value", [float("-inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
def test_rows_without_a_log_sum_exp(size, d, value):
    """A row whose log-sum-exp is -inf (it saw no key) or NaN has no probabilities in any of the kernels: as if its upstream
    gradient were 0."""
    L, Hq, Hkv = 260, 4, 1
    B = batches(L, Hq, Hkv)[size]
    q, segs, d_out = make(1, L, Hq, Hkv, d, (0, L, 0), seed=3900)
    rep = lambda x: bf16_dev(np.repeat(x, B, axis=0))
    qd, kd, vd, dod = rep(q), rep(segs[1].k), rep(segs[1].v), rep(d_out)
    out, dq, dk, dv = (torch.empty_like(x) for x in (qd, qd, kd, vd))
    lse = torch.empty((B, Hq, L), dtype=torch.float32, device=DEV)
    dlm.block_attn(qd, out, block=(kd, vd, 0), lse=lse)
    for i, h in ((0, 0), (33, 1), (40, 3), (L - 1, 2)):
        lse[:, h, i] = value
        d_out[:, i, h] = 0
    ws = torch.empty(dlm.block_attn_bwd_workspace_bytes(B * L, Hq), dtype=torch.uint8, device=DEV)
    dlm.block_attn_bwd(qd, out, dod, lse, dq, block=(kd, vd, 0), d_block=(dk, dv), workspace=ws)
    rq, [(rk, rv)] = obw.attention_backward(q, [segs[1]], d_out)
    for got, ref, bound in zip((dq, dk, dv), (rq, rk, rv), error_bounds(q, [segs[1]], d_out)):
        h = bf16_host(got)
        assert (h == h[:1]).all()
        assert_close(h[:1], ref, bound)
