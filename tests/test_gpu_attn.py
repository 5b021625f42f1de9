"""dlm_block_attn against the oracle, element by element (GPU)."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import KV
from paper_2604_04215_amd import binding as dlm
from paper_2604_04215_amd import synth
from gpu_util import DEV, GuardedWorkspace, attn_rel_err, bf16_dev, bf16_host, dev, rnd

pytestmark = pytest.mark.gpu

TOL = 2e-2          # max relative error, bf16 operands with fp32 accumulation
LSE_TOL = 2e-3


def run_case(B, Lq, Hq, Hkv, d, P, Lb, S, mode="full", bs=0, q_pos0=None, plen=None, variant=0, seed=0,
             block_is_q=True, pos=None, split=None):
    """split: None = no workspace (the call cannot split the keys across workgroups); 0 = a workspace of the size the
    library asks for, split count chosen by the library; n >= 2 = that many splits asked for."""
    q = rnd(seed * 10 + 1, (B, Lq, Hq, d))
    Ltot = P + Lb + S
    k = rnd(seed * 10 + 2, (B, Hkv, Ltot, d))
    v = rnd(seed * 10 + 3, (B, Hkv, Ltot, d))
    q_pos0 = P if q_pos0 is None else q_pos0
    pos = (0, P, P + Lb) if pos is None else pos
    segs = [KV(k[:, :, :P], v[:, :, :P], pos[0]), KV(k[:, :, P:P + Lb], v[:, :, P:P + Lb], pos[1]),
            KV(k[:, :, P + Lb:], v[:, :, P + Lb:], pos[2])]
    ref, ref_lse = oracle.attention(q, segs, mask_mode=mode, bs=bs, q_pos0=q_pos0, prefix_len_b=plen)
    kd, vd, qd = bf16_dev(k), bf16_dev(v), bf16_dev(q)          # one cache tensor: segments are strided views
    out = torch.full((B, Lq, Hq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    lse = torch.full((B, Hq, Lq), float("nan"), dtype=torch.float32, device=DEV)
    dlm.set_option("attn_variant", variant)
    gw = None
    try:
        kw = dict(prefix=(kd[:, :, :P], vd[:, :, :P], pos[0]) if P else None,
                  block=(kd[:, :, P:P + Lb], vd[:, :, P:P + Lb], pos[1]) if Lb else None,
                  suffix=(kd[:, :, P + Lb:], vd[:, :, P + Lb:], pos[2]) if S else None,
                  n_kv_heads=Hkv, mask_mode=dlm.MASK_BLOCK_CAUSAL if mode == "block_causal" else dlm.MASK_FULL,
                  block_size=bs, q_pos0=q_pos0,
                  prefix_len_b=None if plen is None else dev(np.asarray(plen, np.int32)))
        if split is not None:
            dlm.set_option("attn_split", split)
            need = dlm.block_attn_workspace_bytes(qd, **kw)
            assert need % (B * Hq * Lq * (d + 2) * 4) == 0 and need // (B * Hq * Lq * (d + 2) * 4) <= max(split, 16 * (split == 0))
            gw = GuardedWorkspace(need)          # exactly the size asked for, with guard bands
            kw["workspace"] = gw.ws if need else None
        dlm.block_attn(qd, out, lse=lse, **kw)
        torch.cuda.synchronize()
        if gw is not None:
            gw.check()
    finally:
        dlm.set_option("attn_variant", 0)
        dlm.set_option("attn_split", 0)
    err = attn_rel_err(bf16_host(out), ref)
    assert err <= TOL, f"attention rel err {err}"
    got_lse = lse.cpu().numpy().astype(np.float64)
    fin = np.isfinite(ref_lse)
    assert np.array_equal(np.isfinite(got_lse), fin)
    assert np.all(got_lse[~fin] == ref_lse[~fin])
    if fin.any():
        assert np.abs(got_lse[fin] - ref_lse[fin]).max() <= LSE_TOL
    return err


@pytest.mark.parametrize("variant", [0, 1, 2, 3, 8, 9, 10, 12, 13])
def test_rollout_shape_mha(variant):
    # block of 32 against a ragged prefix (several 32-key tiles and a tail), d = 128
    run_case(B=2, Lq=32, Hq=4, Hkv=4, d=128, P=200, Lb=32, S=0, variant=variant, seed=1)


@pytest.mark.parametrize("variant", [0, 2, 3, 4, 5, 6, 7, 11, 13, 14, 15])
def test_dual_cache_and_gqa7(variant):
    # 7 query heads per KV head (224 packed rows), prefix | block | suffix, ragged suffix
    run_case(B=2, Lq=32, Hq=14, Hkv=2, d=128, P=96, Lb=32, S=45, variant=variant, seed=2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Lq,Hq,Hkv", [(1, 2, 2), (5, 4, 2), (32, 4, 4), (40, 6, 2), (70, 4, 1)])
def test_shapes(d, Lq, Hq, Hkv):
    run_case(B=2, Lq=Lq, Hq=Hq, Hkv=Hkv, d=d, P=77, Lb=Lq, S=9, seed=3 + Lq)


@pytest.mark.parametrize("variant", [0, 1, 2, 3, 4, 6, 12, 13, 14, 15])
@pytest.mark.parametrize("bs", [1, 4, 32])
def test_block_causal_rollout(variant, bs):
    # last block(s) of a block-diffusion sequence against the cache; positions are absolute
    run_case(B=2, Lq=8, Hq=8, Hkv=2, d=128, P=188, Lb=8, S=0, mode="block_causal", bs=bs, variant=variant, seed=5)


@pytest.mark.parametrize("variant", [0, 2, 3, 4, 6, 13, 14, 15])
def test_block_causal_full_sequence(variant):
    # training-style pass: Lq = Lk, bidirectional inside blocks of 4, causal across blocks
    B, L, Hq, Hkv, d = 2, 204, 4, 2, 128
    run_case(B=B, Lq=L, Hq=Hq, Hkv=Hkv, d=d, P=0, Lb=L, S=0, mode="block_causal", bs=4, q_pos0=0,
             variant=variant, seed=6)


def test_block_causal_hides_suffix_and_uses_positions():
    # suffix keys lie in later blocks: invisible; shifting every position by a block multiple changes nothing
    run_case(B=1, Lq=8, Hq=4, Hkv=2, d=64, P=40, Lb=8, S=16, mode="block_causal", bs=8, seed=7)
    run_case(B=1, Lq=8, Hq=4, Hkv=2, d=64, P=40, Lb=8, S=16, mode="block_causal", bs=8, q_pos0=1040,
             pos=(1000, 1040, 1048), seed=7)


def test_ragged_prefix_per_sequence():
    run_case(B=3, Lq=32, Hq=4, Hkv=2, d=128, P=100, Lb=32, S=20, plen=[100, 37, 0], seed=8)


@pytest.mark.parametrize("mode,bs", [("full", 0), ("block_causal", 4), ("block_causal", 32)])
@pytest.mark.parametrize("L", [1, 33, 64, 65, 97, 300])
def test_tile_counts_and_two_segments(mode, bs, L):
    # 1, 2, 3, 4 ... key tiles, even and odd counts, ragged tails; one segment and two (full-tile fast path of the
    # loads and stores next to the clamped path of the ragged last tile of each segment)
    run_case(B=1, Lq=L, Hq=4, Hkv=2, d=128, P=0, Lb=L, S=0, mode=mode, bs=bs, q_pos0=0, seed=40 + L)
    run_case(B=2, Lq=40, Hq=2, Hkv=2, d=128, P=L, Lb=40, S=0, mode=mode, bs=bs, seed=41 + L)


def test_degenerate_contexts():
    # no prefix and no suffix; a single key; no key at all (output 0, lse -inf)
    run_case(B=1, Lq=32, Hq=2, Hkv=2, d=128, P=0, Lb=32, S=0, seed=9)
    run_case(B=1, Lq=3, Hq=2, Hkv=1, d=64, P=1, Lb=0, S=0, seed=10)
    run_case(B=2, Lq=4, Hq=2, Hkv=2, d=128, P=5, Lb=0, S=0, plen=[0, 5], seed=11)


def test_noncontiguous_q_and_out_views():
    B, Lq, Hq, Hkv, d, P = 2, 32, 4, 4, 128, 64
    q = rnd(121, (B, Lq, Hq, d))
    k, v = rnd(122, (B, Hkv, P, d)), rnd(123, (B, Hkv, P, d))
    ref, _ = oracle.attention(q, [KV(k, v, 0)])
    big_q = torch.zeros((B, Lq, Hq + 2, d + 64), dtype=torch.bfloat16, device=DEV)
    big_o = torch.zeros_like(big_q)
    qv, ov = big_q[:, :, 1:1 + Hq, :d], big_o[:, :, 1:1 + Hq, :d]
    qv.copy_(bf16_dev(q))
    dlm.block_attn(qv, ov, prefix=(bf16_dev(k), bf16_dev(v), 0))
    torch.cuda.synchronize()
    assert attn_rel_err(bf16_host(ov), ref) <= TOL
    assert float(big_o[:, :, 0].abs().max()) == 0 and float(big_o[..., d:].abs().max()) == 0


def test_rerun_is_bitwise_identical():
    B, Lq, Hq, Hkv, d, P = 2, 32, 8, 2, 128, 300
    q, k, v = bf16_dev(rnd(131, (B, Lq, Hq, d))), bf16_dev(rnd(132, (B, Hkv, P, d))), bf16_dev(rnd(133, (B, Hkv, P, d)))
    o1, o2 = torch.empty_like(q), torch.empty_like(q)
    dlm.block_attn(q, o1, prefix=(k, v, 0))
    dlm.block_attn(q, o2, prefix=(k, v, 0))
    torch.cuda.synchronize()
    assert torch.equal(o1.view(torch.int16), o2.view(torch.int16))


@pytest.mark.parametrize("Lq,Hq,Hkv", [(8, 4, 4), (64, 8, 2)])
def test_peaked_softmax_large_scores(Lq, Hq, Hkv):
    """Scores of magnitude ~50 (Q and K four times the usual scale): nearly one-hot rows, the running maximum
    jumps by far more than the lazy-rescale threshold from tile to tile."""
    B, d, P = 2, 128, 300
    q = synth.f32_to_bf16_bits(np.random.default_rng(3).normal(size=(B, Lq, Hq, d)).astype(np.float32) * 4.0)
    k = synth.f32_to_bf16_bits(np.random.default_rng(4).normal(size=(B, Hkv, P, d)).astype(np.float32) * 4.0)
    v = rnd(305, (B, Hkv, P, d))
    ref, ref_lse = oracle.attention(q, [KV(k, v, 0)])
    out = torch.full((B, Lq, Hq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    lse = torch.full((B, Hq, Lq), float("nan"), dtype=torch.float32, device=DEV)
    dlm.block_attn(bf16_dev(q), out, prefix=(bf16_dev(k), bf16_dev(v), 0), lse=lse)
    torch.cuda.synchronize()
    assert np.abs(ref_lse).max() > 50
    assert attn_rel_err(bf16_host(out), ref) <= TOL
    assert np.abs(lse.cpu().numpy() - ref_lse).max() <= 1e-4 * np.abs(ref_lse).max() + LSE_TOL


def test_non_temporal_kv_stream_changes_nothing():
    """g * Lq <= 32: one workgroup reads its K/V once, with non-temporal loads unless the option turns that off."""
    B, Lq, Hq, Hkv, d, P = 2, 8, 8, 2, 128, 500
    q, k, v = bf16_dev(rnd(141, (B, Lq, Hq, d))), bf16_dev(rnd(142, (B, Hkv, P, d))), bf16_dev(rnd(143, (B, Hkv, P, d)))
    o1, o2 = torch.empty_like(q), torch.empty_like(q)
    dlm.block_attn(q, o1, prefix=(k, v, 0))
    dlm.set_option("attn_nt", 0)
    try:
        dlm.block_attn(q, o2, prefix=(k, v, 0))
    finally:
        dlm.set_option("attn_nt", 1)
    torch.cuda.synchronize()
    assert torch.equal(o1.view(torch.int16), o2.view(torch.int16))
    ref, _ = oracle.attention(rnd(141, (B, Lq, Hq, d)), [KV(rnd(142, (B, Hkv, P, d)), rnd(143, (B, Hkv, P, d)), 0)])
    assert attn_rel_err(bf16_host(o1), ref) <= TOL


@pytest.mark.parametrize("B,Hkv,g,Lq", [(1, 1, 2, 300), (1, 3, 4, 130), (2, 2, 1, 700), (4, 2, 2, 129), (3, 4, 2, 257)])
@pytest.mark.parametrize("variant", [4, 6, 11, 13, 15])
def test_xcd_grouped_grid_covers_every_tile_once(B, Hkv, g, Lq, variant):
    """Group counts 1, 3, 4, 8, 12 (tiles of a group dealt to 8, 8, 2, 1, 2 XCDs) and ragged tile counts, both masks:
    the 1-D grid must produce what the plain (tile, KV head, sequence) grid does, bit for bit, and the oracle's result."""
    d, P = 64, 40
    for mode, bs in (("full", 0), ("block_causal", 8)):
        run_case(B=B, Lq=Lq, Hq=Hkv * g, Hkv=Hkv, d=d, P=P, Lb=Lq, S=0, mode=mode, bs=bs, variant=variant, seed=900 + Lq)
        q = bf16_dev(rnd(9001, (B, Lq, Hkv * g, d)))
        k, v = bf16_dev(rnd(9002, (B, Hkv, Lq, d))), bf16_dev(rnd(9003, (B, Hkv, Lq, d)))
        outs = []
        dlm.set_option("attn_variant", variant)
        try:
            for remap in (7, 1, 0):
                dlm.set_option("attn_remap", remap)
                o = torch.full_like(q, float("nan"))
                dlm.block_attn(q, o, block=(k, v, 0), mask_mode=dlm.MASK_BLOCK_CAUSAL if bs else dlm.MASK_FULL, block_size=bs)
                torch.cuda.synchronize()
                outs.append(o.view(torch.int16))
        finally:
            dlm.set_option("attn_remap", 7)
            dlm.set_option("attn_variant", 0)
        assert torch.equal(outs[0], outs[2]) and torch.equal(outs[1], outs[2])


@pytest.mark.parametrize("Lq,Hq,Hkv,variant", [(32, 4, 4, 0), (8, 8, 2, 0), (130, 4, 2, 0), (130, 4, 2, 11), (300, 2, 1, 6)])
def test_sequences_flagged_inactive_are_skipped(Lq, Hq, Hkv, variant):
    """seq_active[b] == 0: the sequence's rows of out and lse keep what they held; the others match the oracle."""
    B, d, P = 5, 64, 70
    q, k, v = rnd(151, (B, Lq, Hq, d)), rnd(152, (B, Hkv, P + Lq, d)), rnd(153, (B, Hkv, P + Lq, d))
    ref, ref_lse = oracle.attention(q, [KV(k[:, :, :P], v[:, :, :P], 0), KV(k[:, :, P:], v[:, :, P:], P)])
    kd, vd = bf16_dev(k), bf16_dev(v)
    active = np.array([3, 0, 1, 0, -2], np.int32)          # any non-zero value counts as active
    out = torch.full((B, Lq, Hq, d), 7.0, dtype=torch.bfloat16, device=DEV)
    lse = torch.full((B, Hq, Lq), -3.0, dtype=torch.float32, device=DEV)
    dlm.set_option("attn_variant", variant)
    try:
        dlm.block_attn(bf16_dev(q), out, prefix=(kd[:, :, :P], vd[:, :, :P], 0), block=(kd[:, :, P:], vd[:, :, P:], P),
                       lse=lse, seq_active=dev(active))
        torch.cuda.synchronize()
    finally:
        dlm.set_option("attn_variant", 0)
    on = active != 0
    assert attn_rel_err(bf16_host(out)[on], ref[on]) <= TOL
    assert np.abs(lse.cpu().numpy()[on] - ref_lse[on]).max() <= LSE_TOL
    assert bool((out[~torch.from_numpy(on).to(DEV)] == 7.0).all()) and bool((lse[~torch.from_numpy(on).to(DEV)] == -3.0).all())


@pytest.mark.parametrize("variant", [0, 1, 2, 12, 13, 14, 15])
def test_planted_one_hot_values_expose_every_key(variant):
    """V[j] = e_(j mod d): output channel c is the total probability of keys j = c (mod d), so a
    dropped, duplicated or misplaced key shifts some channel by a large relative amount; with Q = 0
    every probability is exactly 1/Lk."""
    B, Lq, Hq, Hkv, d, P, Lb, S = 1, 32, 2, 2, 64, 150, 32, 21
    Lk = P + Lb + S
    v = np.zeros((B, Hkv, Lk, d), np.float32)
    v[:, :, np.arange(Lk), np.arange(Lk) % d] = 1.0
    from paper_2604_04215_amd import synth
    vb = synth.f32_to_bf16_bits(v)
    k = rnd(201, (B, Hkv, Lk, d))
    for qbits in (np.zeros((B, Lq, Hq, d), np.uint16), rnd(202, (B, Lq, Hq, d), 0.3)):
        segs = [KV(k[:, :, :P], vb[:, :, :P], 0), KV(k[:, :, P:P + Lb], vb[:, :, P:P + Lb], P),
                KV(k[:, :, P + Lb:], vb[:, :, P + Lb:], P + Lb)]
        ref, _ = oracle.attention(qbits, segs)
        kd, vd = bf16_dev(k), bf16_dev(vb)
        out = torch.empty((B, Lq, Hq, d), dtype=torch.bfloat16, device=DEV)
        dlm.set_option("attn_variant", variant)
        try:
            dlm.block_attn(bf16_dev(qbits), out, prefix=(kd[:, :, :P], vd[:, :, :P], 0),
                           block=(kd[:, :, P:P + Lb], vd[:, :, P:P + Lb], P),
                           suffix=(kd[:, :, P + Lb:], vd[:, :, P + Lb:], P + Lb))
            torch.cuda.synchronize()
        finally:
            dlm.set_option("attn_variant", 0)
        from paper_2604_04215_amd.synth import bf16_bits_to_f64
        got = bf16_bits_to_f64(bf16_host(out))
        # every channel is a sum of 3-4 probabilities: a per-element relative check is meaningful here
        assert np.abs(got - ref).max() <= 2e-2 * ref.min()


def test_prefix_only_cache_with_block_and_suffix_queries():
    """Prefix-only caching: only the prompt and finished blocks are cached, and the step recomputes the current
    block AND the still-masked suffix, so the query set is block + suffix (Lq = Lb + S) against
    [cached prefix | those same Lb + S fresh rows].  Same kernel, larger Lq."""
    for Lb, S, P in [(32, 96, 200), (32, 224, 72)]:
        run_case(B=2, Lq=Lb + S, Hq=4, Hkv=2, d=128, P=P, Lb=Lb + S, S=0, seed=77 + S)


def test_largest_batch_the_grid_takes():
    """B = 65535 (the launch grid's limit; one more is refused): one query row, one key, per sequence."""
    B, d = 65535, 64
    q, k, v = rnd(991, (B, 1, 1, d)), rnd(992, (B, 1, 1, d)), rnd(993, (B, 1, 1, d))
    out = torch.full((B, 1, 1, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    dlm.block_attn(bf16_dev(q), out, block=(bf16_dev(k), bf16_dev(v), 0))
    torch.cuda.synchronize()
    got = synth.bf16_bits_to_f64(bf16_host(out)).reshape(B, d)
    assert np.array_equal(got, synth.bf16_bits_to_f64(v).reshape(B, d))        # softmax over one key: O = V exactly
    big = torch.zeros((65536, 1, 1, d), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(dlm.DlmError):
        dlm.block_attn(big, big.clone(), block=(big.view(65536, 1, 1, d), big.view(65536, 1, 1, d), 0))


# ---- key split across workgroups + merge kernel ------------------------------------------------------------
@pytest.mark.parametrize("variant", [0, 1, 12, 8])
@pytest.mark.parametrize("split", [2, 3, 5])
def test_key_split_rollout_shape(variant, split):
    """One workgroup per (sequence, KV head) split into `split` workgroups over the key tiles: ragged prefix (a tail
    tile), block and suffix segments, d = 128 and 64; every element against the oracle."""
    run_case(B=2, Lq=32, Hq=4, Hkv=4, d=128, P=712, Lb=32, S=100, variant=variant, seed=41, split=split)
    run_case(B=3, Lq=16, Hq=4, Hkv=2, d=64, P=1000, Lb=16, S=0, variant=variant, seed=42, split=split)


@pytest.mark.parametrize("variant", [0, 2, 3, 4, 6, 11, 13, 14, 15])
@pytest.mark.parametrize("split", [2, 3])
def test_key_split_row_tile_shapes(variant, split):
    """128- / 256-row workgroups (7 heads per KV head x 32 rows = 224 rows, two ragged row tiles) with the keys split
    across workgroups, full and block-causal masks, plain and XCD-grouped grids."""
    run_case(B=2, Lq=32, Hq=14, Hkv=2, d=128, P=640, Lb=32, S=0, variant=variant, seed=43, split=split)
    run_case(B=1, Lq=160, Hq=4, Hkv=2, d=128, P=96, Lb=160, S=0, mode="block_causal", bs=32, q_pos0=96, variant=variant,
             seed=44, split=split)
    dlm.set_option("attn_remap", 0)
    try:
        run_case(B=2, Lq=40, Hq=8, Hkv=2, d=64, P=520, Lb=40, S=30, variant=variant, seed=45, split=split)
    finally:
        dlm.set_option("attn_remap", 7)


def test_key_split_edge_cases():
    """More splits than a sequence has key tiles (some workgroups get none), sequences whose prefix is empty, rows
    that see no key at all, and a split count the library lowers because the problem has few tiles."""
    # ragged per-sequence prefix: sequence 1 has no prefix at all, sequence 2 a single key
    run_case(B=3, Lq=32, Hq=2, Hkv=2, d=128, P=640, Lb=32, S=0, plen=[640, 0, 1], variant=1, seed=46, split=5)
    run_case(B=3, Lq=32, Hq=2, Hkv=2, d=128, P=640, Lb=32, S=0, plen=[640, 0, 1], variant=4, seed=46, split=4)
    # block-causal where early rows see only the first keys: splits past their visible range hold nothing for them
    run_case(B=1, Lq=64, Hq=2, Hkv=1, d=128, P=0, Lb=640, S=0, mode="block_causal", bs=4, q_pos0=0, variant=1, seed=47, split=4)
    run_case(B=1, Lq=256, Hq=2, Hkv=1, d=128, P=0, Lb=640, S=0, mode="block_causal", bs=4, q_pos0=0, variant=6, seed=47, split=4)
    # few tiles: the library lowers the split count (at least four tiles per workgroup) or drops the split
    run_case(B=1, Lq=32, Hq=2, Hkv=2, d=64, P=100, Lb=32, S=0, variant=0, seed=48, split=6)
    # library-chosen split: 16 workgroups unsplit and 64 key tiles -> 16 splits of 4 tiles; 8 of 128 rows -> 16 splits
    run_case(B=2, Lq=32, Hq=8, Hkv=8, d=128, P=2016, Lb=32, S=0, variant=0, seed=49, split=0)
    run_case(B=1, Lq=32, Hq=32, Hkv=8, d=128, P=2080, Lb=32, S=0, variant=0, seed=50, split=0)
    q = torch.zeros((2, 32, 8, 128), dtype=torch.bfloat16, device=DEV)
    k = torch.zeros((2, 8, 2048, 128), dtype=torch.bfloat16, device=DEV)
    assert dlm.block_attn_workspace_bytes(q, block=(k, k, 0)) == 16 * 2 * 8 * 32 * 130 * 4
    assert dlm.block_attn_workspace_bytes(q, block=(k[:, :, :992], k[:, :, :992], 0)) == 0      # 31 tiles: too few to pay


def test_key_split_is_deterministic_and_skips_inactive_sequences():
    B, Lq, H, d, P = 4, 32, 4, 128, 800
    q = bf16_dev(rnd(5001, (B, Lq, H, d)))
    k, v = bf16_dev(rnd(5002, (B, H, P + Lq, d))), bf16_dev(rnd(5003, (B, H, P + Lq, d)))
    kw = dict(prefix=(k[:, :, :P], v[:, :, :P], 0), block=(k[:, :, P:], v[:, :, P:], P))
    dlm.set_option("attn_split", 3)
    try:
        ws = torch.empty(dlm.block_attn_workspace_bytes(q, **kw), dtype=torch.uint8, device=DEV)
        assert ws.numel() == 3 * B * H * Lq * (d + 2) * 4
        outs = []
        for _ in range(2):
            ws.fill_(0xFF)                                   # whatever the workspace held before must not matter
            o = torch.full_like(q, float("nan"))
            lse = torch.full((B, H, Lq), float("nan"), device=DEV)
            dlm.block_attn(q, o, lse=lse, workspace=ws, **kw)
            torch.cuda.synchronize()
            outs.append((o.view(torch.int16).clone(), lse.clone()))
        assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
        # unsplit result: same values up to the rounding of a different summation order
        dlm.set_option("attn_split", 1)
        o1 = torch.full_like(q, float("nan"))
        dlm.block_attn(q, o1, workspace=ws, **kw)
        torch.cuda.synchronize()
        assert (outs[0][0].view(torch.bfloat16).float() - o1.float()).abs().max().item() <= 2e-2
        # sequences 1 and 3 inactive: their rows keep the sentinel, the others equal the full run
        dlm.set_option("attn_split", 3)
        act = dev(np.array([1, 0, 5, 0], np.int32))
        o2 = torch.full_like(q, 7.0)
        dlm.block_attn(q, o2, workspace=ws, seq_active=act, **kw)
        torch.cuda.synchronize()
        assert torch.equal(o2.view(torch.int16)[[0, 2]], outs[0][0][[0, 2]])
        assert (o2[[1, 3]] == 7.0).all().item()
        # a workspace that is too small: the call runs unsplit instead of failing
        o3 = torch.full_like(q, float("nan"))
        dlm.block_attn(q, o3, workspace=ws[:1024], **kw)
        torch.cuda.synchronize()
        assert torch.equal(o3.view(torch.int16), o1.view(torch.int16))
    finally:
        dlm.set_option("attn_split", 0)


@pytest.mark.parametrize("variant", [13, 14, 15])
def test_two_key_groups_per_workgroup_edge_cases(variant):
    """128-row workgroups whose eight wavefronts form two key groups: odd tile counts (the second group's last tile
    does not exist), a single tile, ragged per-sequence prefixes down to none, d = 64, rows that see nothing."""
    run_case(B=3, Lq=32, Hq=4, Hkv=2, d=128, P=100, Lb=32, S=20, plen=[100, 37, 0], variant=variant, seed=61)
    run_case(B=1, Lq=130, Hq=2, Hkv=1, d=64, P=0, Lb=20, S=0, variant=variant, seed=62)            # one tile only
    run_case(B=2, Lq=70, Hq=6, Hkv=2, d=64, P=333, Lb=70, S=11, variant=variant, seed=63)
    run_case(B=1, Lq=200, Hq=2, Hkv=1, d=128, P=0, Lb=200, S=0, mode="block_causal", bs=4, q_pos0=0, variant=variant, seed=64)
    run_case(B=2, Lq=4, Hq=2, Hkv=2, d=128, P=5, Lb=0, S=0, plen=[0, 5], variant=variant, seed=65)


@pytest.mark.parametrize("d,bs,packed", [(64, 0, False), (64, 4, False), (128, 0, False), (128, 32, False), (64, 4, True), (128, 0, True)])
def test_launches_deep_enough_for_issue_priorities(d, bs, packed):
    """3 * 768 * 128 and more rows with 768 and more keys (packed: a mean length of 512) run the kernel with issue priorities: bit for bit
    what two launches of half the batch give, which are too small for it."""
    H, B, Lq, Lk = 4, 568, 130, 768
    mode = dict(mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=bs) if bs else {}
    g = torch.Generator(device=DEV).manual_seed(d + bs)
    rn = lambda *shape: torch.randn(shape, generator=g, device=DEV).bfloat16()
    if packed:
        lens = np.where(np.arange(148) % 2, 417, 607)
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        T, half = int(cu[-1]), int(cu[74])
        assert H * T >= 3 * 768 * 128 > H * half and T // 148 == 512
        q, k, v = rn(T, H, d), rn(T, H, d), rn(T, H, d)
        run = lambda q, k, v, o, c: dlm.varlen_attn(q, k, v, o, dev(c), 607, **mode)
        parts = [(slice(0, half), cu[:75]), (slice(half, T), cu[74:] - cu[74])]
        whole = cu
    else:
        q, k, v = rn(B, Lq, H, d), rn(B, H, Lk, d), rn(B, H, Lk, d)
        run = lambda q, k, v, o, c: dlm.block_attn(q, o, block=(k, v, 0), q_pos0=Lk - Lq, **mode)
        parts, whole = [(slice(0, B // 2), None), (slice(B // 2, B), None)], None
    out, ref = torch.zeros_like(q), torch.zeros_like(q)
    run(q, k, v, out, whole)
    for part, c in parts:
        run(q[part], k[part], v[part], ref[part], c)
    assert out.any() and torch.equal(out.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("d,Lq,Hq,Hkv,P,S,split,kw", [
    (64, 1, 33, 1, 0, 0, 0, {}),                              # one key: seven of the eight wavefronts have no tile
    (128, 33, 2, 2, 190, 7, 0, {}),                           # 9 tiles over three segments, a row tile of one row
    (64, 40, 7, 1, 225, 0, 0, dict(mode="block_causal", bs=8)),
    (128, 20, 8, 2, 250, 0, 0, dict(plen=[250, 31])),         # a sequence whose prefix is one tile
    (128, 32, 8, 2, 1500, 0, 5, {}),                          # splits of nine and ten tiles
    (64, 32, 14, 2, 1030, 0, 16, dict(mode="block_causal", bs=32)),
])
def test_eight_wavefronts_that_share_the_keys_of_32_rows(d, Lq, Hq, Hkv, P, S, split, kw):
    run_case(B=2, Lq=Lq, Hq=Hq, Hkv=Hkv, d=d, P=P, Lb=Lq, S=S, seed=60 + P, variant=16, split=split, **kw)


@pytest.mark.parametrize("B,Lq,Hq,Hkv,d,P,kw", [
    (1, 32, 4, 4, 64, 2016, {}), (24, 16, 4, 4, 64, 1000, {}), (24, 16, 4, 4, 64, 2016, {}),   # up to 32 rows: splits of 8 tiles, none, 2
    (1, 32, 32, 8, 128, 1000, {}), (2, 32, 28, 4, 128, 1100, {}), (4, 32, 28, 4, 128, 1100, {}),   # splits of 32-row workgroups, none
    (6, 32, 14, 2, 64, 2100, dict(mode="block_causal", bs=32)),   # as many splits as the fullest XCD has CUs for
    (8, 32, 28, 4, 128, 2900, {}), (8, 32, 28, 4, 128, 2000, {}),   # more tiles than 32-row workgroups are worth, and fewer
])
def test_splits_that_a_call_takes_of_those_it_has_room_for(B, Lq, Hq, Hkv, d, P, kw):
    """Calls with a workspace for the most splits: how many of them are taken, and the rows of a workgroup, follow from the shape."""
    run_case(B=B, Lq=Lq, Hq=Hq, Hkv=Hkv, d=d, P=P, Lb=Lq, S=0, seed=70 + B, split=0, **kw)


@pytest.mark.parametrize("B,L,Hq,Hkv,d,bs", [(1, 1008, 16, 2, 128, 16), (2, 500, 14, 2, 64, 4), (3, 800, 28, 4, 128, 0), (1, 900, 4, 4, 64, 0),
                                             (1, 2050, 4, 4, 64, 8), (6, 348, 4, 4, 64, 32)])
def test_full_sequences_on_both_sides_of_the_lines_between_shapes(B, L, Hq, Hkv, d, bs):
    run_case(B=B, Lq=L, Hq=Hq, Hkv=Hkv, d=d, P=0, Lb=L, S=0, seed=80 + L, **(dict(mode="block_causal", bs=bs, q_pos0=0) if bs else {}))


def planned_and_named(call, out, **named):
    """A call as planned and with its shape (and split) by name: the same kernel, so the same bits."""
    call()
    planned = out.clone()
    out.zero_()
    for name, value in named.items():
        dlm.set_option(name, value)
    try:
        call()
    finally:
        for name in named:
            dlm.set_option(name, 0)
    assert planned.any() and torch.equal(planned.view(torch.int16), out.view(torch.int16))


def normal(seed, *shape):
    return torch.randn(shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV, dtype=torch.bfloat16)


@pytest.mark.parametrize("B,L,Hq,Hkv,d,variant", [
    (4, 500, 32, 32, 128, 4), (2, 1000, 32, 32, 128, 4), (16, 1500, 4, 4, 64, 6),   # a CU would get too much of them one after another
    (1, 1500, 16, 2, 128, 13), (2, 600, 32, 8, 128, 13), (10, 1300, 4, 4, 64, 13),   # the longest is what the launch waits for
    (-16, 533, 16, 2, 128, 6), (-8, 1000, 16, 2, 128, 6), (-4, 1600, 16, 2, 64, 13), (-6, 1250, 8, 2, 128, 13), (-11, 620, 1, 1, 128, 11),   # packed: lengths from 1 to L
])
def test_eight_wavefronts_under_a_causal_mask_where_the_longest_decides(B, L, Hq, Hkv, d, variant):
    mask = dict(mask_mode=dlm.MASK_BLOCK_CAUSAL, block_size=32)
    if B > 0:
        q, k, v = normal(1, B, L, Hq, d), normal(2, B, Hkv, L, d), normal(3, B, Hkv, L, d)
        out = torch.zeros_like(q)
        planned_and_named(lambda: dlm.block_attn(q, out, block=(k, v, 0), **mask), out, attn_variant=variant)
    else:
        lens = np.linspace(1, L, -B).astype(np.int32)
        cu = dev(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
        T = int(lens.sum())
        q, k, v = normal(1, T, Hq, d), normal(2, T, Hkv, d), normal(3, T, Hkv, d)
        out = torch.zeros_like(q)
        planned_and_named(lambda: dlm.varlen_attn(q, k, v, out, cu, L, **mask), out, attn_variant=variant)


KERNEL_NAMES = """
import json, sys
import torch
from torch.profiler import ProfilerActivity, profile
from paper_2604_04215_amd import binding as dlm
for B, L, Hq, Hkv, bs in json.loads(sys.argv[1]):
    q, k = (torch.ones(B, *s, 128, device="cuda:0", dtype=torch.bfloat16) for s in ((L, Hq), (Hkv, L)))
    out = torch.zeros_like(q)
    call = lambda: dlm.block_attn(q, out, block=(k, k, 0), mask_mode=dlm.MASK_BLOCK_CAUSAL if bs else dlm.MASK_FULL, block_size=bs)
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    print("NAME", next(e.name for e in prof.events() if "attn_kernel<" in e.name), flush=True)
"""


def test_workgroups_a_cu_for_less_than_768():
    """Two or three workgroups a CU give the same bits: the shape is read from the kernel's name (in a process of its own, which a profiler follows)."""
    cases = [(6, 2000, 8, 2, 4, 2), (4, 1300, 16, 8, 4, 2),                             # causal, 25 - 64 key tiles: two
             (12, 420, 16, 8, 4, 3), (16, 640, 8, 4, 32, 3), (19, 264, 16, 2, 32, 3), (4, 2600, 8, 8, 32, 3),   # fewer, more: three
             (3, 800, 28, 4, 0, 3), (3, 3000, 8, 2, 0, 3)]                              # and without a mask
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", KERNEL_NAMES, json.dumps([c[:5] for c in cases])], cwd=root, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr[-2000:]
    names = [line for line in run.stdout.splitlines() if line.startswith("NAME")]
    for name, case in zip(names, cases, strict=True):
        row_waves, key_waves, tiles, causal, _, a_cu = name.split("attn_kernel<128, ")[1].split(">")[0].split(", ")[:6]
        assert (row_waves, key_waves, tiles, causal, a_cu) == ("4", "1", "1", "true" if case[4] else "false", str(case[5])), (case, name)


@pytest.mark.parametrize("B,Lb,Hq,Hkv,d,P,variant,split", [
    (20, 16, 14, 2, 64, 8000, 13, 6), (5, 64, 16, 2, 64, 12000, 13, 6), (20, 48, 4, 4, 128, 8000, 13, 3),   # too few 32-row workgroups for keys that long
    (18, 64, 7, 1, 64, 3891, 13, 3), (25, 64, 4, 4, 128, 4577, 13, 2), (31, 8, 16, 2, 128, 7963, 13, 4),    # more than one a CU; keys read on two XCDs
    (4, 32, 14, 2, 64, 4000, 16, 4), (4, 32, 8, 2, 128, 2000, 16, 8), (1, 32, 32, 8, 128, 8000, 16, 8), (7, 32, 16, 2, 128, 2237, 16, 2),   # but enough here
    (1, 4, 4, 4, 128, 4000, 12, 16), (2, 4, 14, 2, 64, 3000, 12, 12), (8, 4, 4, 4, 64, 1300, 12, 6), (1, 16, 28, 4, 128, 4000, 16, 16),   # no split of nine tiles
    (40, 16, 16, 2, 64, 289, 11, 1), (63, 16, 16, 2, 64, 289, 13, 1),   # two 32-row workgroups a CU; and keys read on four XCDs for them
])
def test_rows_of_a_split(B, Lb, Hq, Hkv, d, P, variant, split):
    q, k, v = normal(1, B, Lb, Hq, d), normal(2, B, Hkv, P + Lb, d), normal(3, B, Hkv, P + Lb, d)
    segs = dict(prefix=(k[:, :, :P], v[:, :, :P], 0), block=(k[:, :, P:], v[:, :, P:], P))
    ws = torch.empty(16 * B * Lb * Hq * (d + 2) * 4, dtype=torch.uint8, device=DEV)
    out = torch.zeros_like(q)
    planned_and_named(lambda: dlm.block_attn(q, out, workspace=ws, **segs), out, attn_variant=variant, attn_split=split)


@pytest.mark.parametrize("B,Lq,Hq,Hkv,d,L,most,used", [(1, 32, 4, 4, 64, 2048, 16, 8), (4, 32, 8, 2, 128, 2000, 15, 8), (1, 16, 28, 4, 128, 2000, 15, 8)])
def test_a_workspace_for_the_splits_that_a_call_takes(B, Lq, Hq, Hkv, d, L, most, used):
    """dlm_block_attn_workspace_bytes covers every number of splits; a buffer for those that the call takes is enough, 16 bytes less are not."""
    q, k, v = normal(1, B, Lq, Hq, d), normal(2, B, Hkv, L, d), normal(3, B, Hkv, L, d)
    segs, split = dict(block=(k, v, 0)), B * Lq * Hq * (d + 2) * 4
    assert dlm.block_attn_workspace_bytes(q, **segs) == most * split
    outs = []
    for size in (most * split, used * split, used * split - 16, 0):
        gw = GuardedWorkspace(size) if size else None
        out = torch.zeros_like(q)
        dlm.block_attn(q, out, workspace=gw and gw.ws, **segs)
        torch.cuda.synchronize()
        if gw:
            gw.check()
        outs.append(out.view(torch.int16))
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[2], outs[3]) and not torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("B,L,Hq,Hkv,d,variant", [
    (32, 48, 8, 4, 64, 13), (5, 48, 32, 32, 64, 13), (7, 75, 16, 2, 64, 11), (3, 100, 28, 4, 64, 11),   # 257 - 512 of 32 rows: two key tiles, three, four
    (17, 132, 7, 1, 64, 13), (10, 112, 14, 2, 64, 13),                          # more than two of them a CU on the fullest XCD
    (5, 100, 16, 2, 128, 13), (5, 100, 8, 1, 128, 11),                          # 35 of them on the fullest XCD, 20
])
def test_short_sequences_on_few_rows(B, L, Hq, Hkv, d, variant):
    q, k, v = normal(1, B, L, Hq, d), normal(2, B, Hkv, L, d), normal(3, B, Hkv, L, d)
    out = torch.zeros_like(q)
    planned_and_named(lambda: dlm.block_attn(q, out, block=(k, v, 0)), out, attn_variant=variant)
