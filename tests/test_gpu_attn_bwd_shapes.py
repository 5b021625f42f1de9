"""Every shape of the backward kernels at the sizes where it can go wrong: keys and rows around a wavefront's 64 and a workgroup's
128, group sizes that do and do not divide a 32-row tile, token strides that do not fit 32-bit offsets.  The batch decides which
shape runs: 1 sequence takes the row-split dK / dV kernel, more than 256 slabs of 128 keys the key-split one, 1024 workgroups of
128 rows and more (d = 128) the 64-row dQ kernel.  All sequences of a batch are copies of one, so the first is checked against the oracle
and the others have to have its bits."""
import numpy as np
import pytest
import torch

from oracle import KV
from oracle import backward as obw
from paper_2604_04215_amd import binding as dlm
from paper_2604_04215_amd import synth
from gpu_util import DEV, bf16_dev, bf16_host
from test_gpu_attn_bwd import FRO_TOL, TOL, fro_err, make, run_bwd

pytestmark = pytest.mark.gpu


def batches(L, Hq, Hkv):
    slabs, rows = (L + 127) // 128 * Hkv, (L * (Hq // Hkv) + 127) // 128 * Hkv
    return [1, 256 // slabs + 1, (1024 + rows - 1) // rows]


def elem_err(got_u16, ref):
    """max |got - ref| / max(|ref|, rms of the reference tensor).  Not the row's rms: where a row sees a few keys and one takes nearly
    all of the probability, its exact gradient vanishes (dS = P (dP - delta), dP -> delta) while delta, formed from the bf16
    output, keeps an error of up to 2^-9 sum_c |dO_c O_c|; that error is small against the tensor, not against such a row."""
    got = synth.bf16_bits_to_f64(got_u16).reshape(ref.shape)
    den = np.maximum(np.abs(ref), np.sqrt((ref ** 2).mean()))
    return float((np.abs(got - ref) / np.where(den == 0, 1.0, den)).max())   # (one key: the exact gradient is 0)


def check_copies(q, segs, d_out, B, mode="full", bs=0):
    rep = lambda x: np.repeat(x, B, axis=0)
    dq, grads = run_bwd(rep(q), [None if s is None else KV(rep(s.k), rep(s.v), s.pos0, s.rule) for s in segs], rep(d_out), mode=mode, bs=bs)
    rdq, rg = obw.attention_backward(q, [s for s in segs if s is not None], d_out, mask_mode=mode, bs=bs)
    pairs = [(dq, rdq)] + [(got, ref) for g, r in zip([g for g in grads if g is not None], rg) for got, ref in zip(g, r)]
    for got, ref in pairs:
        assert (got == got[:1]).all()
        assert elem_err(got[:1], ref) <= TOL and fro_err(got[:1], ref) <= FRO_TOL


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


@pytest.mark.parametrize("B", [16, 32], ids=["row-split", "key-split"])
def test_paired_slabs(B):
    """33 slabs of 64 keys (17 of 128), 1024 of them and more: the launch pairs the slabs of a block-causal segment.  The gradients
    against the same sequence by itself (no pairs): two bf16 results whose sums over rows differ in order."""
    q, segs, d_out = make(1, 2100, 2, 2, 64, (0, 2100, 0), seed=3600)
    rep = lambda x: np.repeat(x, B, axis=0)
    dq, grads = run_bwd(rep(q), [None, KV(rep(segs[1].k), rep(segs[1].v), 0), None], rep(d_out), mode="block_causal", bs=32)
    dq1, grads1 = run_bwd(q, segs, d_out, mode="block_causal", bs=32)
    for a, r in ((dq, dq1), (grads[1][0], grads1[1][0]), (grads[1][1], grads1[1][1])):
        assert (a == a[:1]).all()
        assert fro_err(a[:1], synth.bf16_bits_to_f64(r).reshape(r.shape)) <= FRO_TOL


@pytest.mark.parametrize("what", ["q", "kv"])
@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
def test_strides_beyond_32_bit_offsets(size, what):
    """Token strides of 2^23 elements (2^24 bytes) and more leave the 32-bit offsets of the tile requests."""
    L, Hq, Hkv, d, st = 40, 3, 1, 128, (1 << 23) + 8
    B = batches(L, Hq, Hkv)[size]
    q, segs, d_out = make(1, L, Hq, Hkv, d, (0, L, 0), seed=3700)

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
    dlm.block_attn(qd, out, block=(kd, vd, 0), lse=lse)
    dq = torch.empty_like(out)
    ws = torch.empty(dlm.block_attn_bwd_workspace_bytes(B * L, Hq), dtype=torch.uint8, device=DEV)
    dlm.block_attn_bwd(qd, out, dod, lse, dq, block=(kd, vd, 0), d_block=(dk, dv), workspace=ws)
    rq, [(rk, rv)] = obw.attention_backward(q, [segs[1]], d_out)
    for got, ref in ((dq, rq), (dk, rk), (dv, rv)):
        h = bf16_host(got.contiguous())
        assert (h == h[:1]).all()
        assert elem_err(h[:1], ref) <= TOL and fro_err(h[:1], ref) <= FRO_TOL


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
    for got, ref in ((dq[:, :, heads], rq), (dk, rk), (dv, rv)):
        assert elem_err(bf16_host(got), ref) <= TOL and fro_err(bf16_host(got), ref) <= FRO_TOL


@pytest.mark.parametrize("value", [float("-inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("size", [0, 1, 2], ids=["row-split", "key-split", "dq64"])
def test_rows_without_a_log_sum_exp(size, d, value):
    """A row whose log-sum-exp is -inf (it saw no key) or NaN has no probabilities in any of the kernels: as if its upstream
    gradient were 0."""
    L, Hq, Hkv = 70, 4, 1
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
    for got, ref in ((dq, rq), (dk, rk), (dv, rv)):
        h = bf16_host(got)
        assert (h == h[:1]).all()
        assert elem_err(h[:1], ref) <= TOL and fro_err(h[:1], ref) <= FRO_TOL
