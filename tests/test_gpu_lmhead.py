"""dlm_lmhead_confidence against the oracle (GPU)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_04215_amd import binding as dlm
from paper_2604_04215_amd import synth
from gpu_util import DEV, GuardedWorkspace, bf16_dev, dev, rnd

pytestmark = pytest.mark.gpu

CONF_TOL = 1e-3     # absolute, confidences
MARGIN = 1e-3       # rows whose top-2 logit margin is below this may legitimately pick the other token
Z_TOL = 2e-3        # logits-scale outputs (lse, zmax, z2nd): fp32 accumulation over Dh terms


def run_lm(hidden, w, *, row_idx=None, M=None, m_dev=None, forbid=-1, inv_t=1.0, scatter=False, target=None,
           M_expected=0):
    R, Dh = hidden.shape
    V = w.shape[0]
    hd, wd = bf16_dev(hidden), bf16_dev(w)
    ridx = None if row_idx is None else dev(np.asarray(row_idx, np.int32))
    Mh = M if M is not None else (len(row_idx) if row_idx is not None else R)
    n_out = R if scatter else Mh
    f = lambda: torch.full((n_out,), float("nan"), dtype=torch.float32, device=DEV)
    conf, lse, zmax, z2nd = f(), f(), f(), f()
    tok = torch.full((n_out,), -7, dtype=torch.int32, device=DEV)
    tgt = zt = None
    if target is not None:
        tgt, zt = dev(np.asarray(target, np.int32)), f()
    gw = GuardedWorkspace(dlm.lmhead_workspace_bytes(Mh, V))     # exactly the size the library asks for, guarded
    dlm.lmhead_confidence(hd, wd, conf, tok, M=Mh, row_idx=ridx,
                          m_dev=None if m_dev is None else dev(np.asarray([m_dev], np.int32)),
                          forbid_token=forbid, inv_temperature=inv_t, out_scatter=scatter,
                          lse=lse, zmax=zmax, z2nd=z2nd, target=tgt, ztarget=zt, workspace=gw.ws,
                          M_expected=M_expected)
    gw.check()
    out = dict(conf=conf.cpu().numpy(), tok=tok.cpu().numpy(), lse=lse.cpu().numpy(), zmax=zmax.cpu().numpy(),
               z2nd=z2nd.cpu().numpy())
    if zt is not None:
        out["zt"] = zt.cpu().numpy()
    return out


def compare_prefix(got, ref, m):
    """The first m outputs against the oracle's; the rest must be untouched.  Few rows: confidences only."""
    if m >= 20:
        compare({k: v[:m] for k, v in got.items()}, {k: v[:m] for k, v in ref.items() if k != "zt"})
    elif m > 0:
        assert np.abs(got["conf"][:m].astype(np.float64) - ref["conf"][:m]).max() <= CONF_TOL
        assert np.abs(got["lse"][:m] - ref["lse"][:m]).max() <= Z_TOL
    assert np.all(np.isnan(got["conf"][m:])) and np.all(got["tok"][m:] == -7)


def compare(got, ref, sel=None):
    """got arrays indexed by output slot; ref from the oracle in the same order (sel picks got's slots)."""
    g = {k: (v if sel is None else v[sel]) for k, v in got.items()}
    assert np.abs(g["conf"].astype(np.float64) - ref["conf"]).max() <= CONF_TOL
    margin = ref["zmax"] - ref["z2nd"]
    clear = margin >= MARGIN
    assert np.array_equal(g["tok"][clear], ref["tok"][clear])
    assert clear.mean() > 0.9
    assert np.abs(g["lse"] - ref["lse"]).max() <= Z_TOL
    assert np.abs(g["zmax"] - ref["zmax"]).max() <= Z_TOL
    both = np.isfinite(ref["z2nd"])
    assert np.abs(g["z2nd"][both] - ref["z2nd"][both]).max() <= Z_TOL
    if "zt" in ref:
        fin = np.isfinite(ref["zt"])
        assert np.abs(g["zt"][fin] - ref["zt"][fin]).max() <= Z_TOL
        assert np.array_equal(np.isfinite(g["zt"]), fin)


@pytest.mark.parametrize("M,Dh,V", [(1, 64, 300), (16, 256, 2048), (33, 128, 777), (64, 192, 1000), (90, 128, 600),
                                    (100, 320, 1500), (150, 128, 700), (200, 256, 900), (256, 128, 2048),
                                    (300, 64, 515), (700, 64, 400)])
def test_shapes_vs_oracle(M, Dh, V):
    # covers every row-tile variant (<=32, <=64, <=128, <=256 rows), several row chunks, ragged V tails
    h, w = rnd(M + Dh, (M, Dh)), rnd(V + Dh, (V, Dh), Dh ** -0.25)
    ref = oracle.lmhead(h, w, forbid_token=V - 1)
    got = run_lm(h, w, forbid=V - 1)
    compare(got, ref)
    assert np.all(got["tok"] != V - 1)


@pytest.mark.parametrize("variant", range(30))
def test_every_kernel_shape(variant):
    # each entry of the library's shape table on a problem with several row chunks and ragged tails
    M, Dh, V = 300, 192, 1100
    h, w = rnd(900, (M, Dh)), rnd(901, (V, Dh), Dh ** -0.25)
    tgt = np.random.default_rng(2).integers(0, V, size=M).astype(np.int32)
    ref = oracle.lmhead(h, w, forbid_token=V - 1, target=tgt)
    dlm.set_option("lmhead_variant", variant)
    try:
        got = run_lm(h, w, forbid=V - 1, target=tgt)
    finally:
        dlm.set_option("lmhead_variant", -1)
    compare(got, ref)


@pytest.mark.parametrize("variant", list(range(10, 24)) + [27])
@pytest.mark.parametrize("Dh", [640, 704])
def test_ring_shapes_reach_their_steady_state_loop(variant, Dh):
    # the direct-to-LDS shapes run prologue + drain only while Dh < 7 stages of 32: here 20 and 22 stages
    M, V = 270, 600
    h, w = rnd(910 + Dh, (M, Dh)), rnd(911 + Dh, (V, Dh), Dh ** -0.25)
    ref = oracle.lmhead(h, w, forbid_token=3)
    dlm.set_option("lmhead_variant", variant)
    try:
        got = run_lm(h, w, forbid=3)
    finally:
        dlm.set_option("lmhead_variant", -1)
    compare(got, ref)


@pytest.mark.parametrize("variant,M", [(0, 413), (1, 413), (20, 2806), (21, 2900), (3, 1400)])
def test_row_chunk_counts_without_a_divisor(variant, M):
    # 13 / 7 / 11 / 12 row chunks: counts that are prime or have only a small divisor, so the blocks of row chunks that an
    # XCD runs side by side degenerate (one chunk per block, or blocks that do not fill the XCD)
    Dh, V = 128, 600
    h, w = rnd(940 + M, (M, Dh)), rnd(941 + M, (V, Dh), Dh ** -0.25)
    ref = oracle.lmhead(h, w, forbid_token=V - 1)
    dlm.set_option("lmhead_variant", variant)
    try:
        got = run_lm(h, w, forbid=V - 1)
    finally:
        dlm.set_option("lmhead_variant", -1)
    compare(got, ref)


def test_gather_scatter_mdev_temperature_target():
    R, Dh, V = 96, 128, 1000
    h, w = rnd(1, (R, Dh)), rnd(2, (V, Dh), Dh ** -0.25)
    idx = np.array(sorted(np.random.default_rng(0).permutation(R)[:41]), np.int32)
    tgt_dense = np.random.default_rng(1).integers(0, V, size=R).astype(np.int32)
    ref = oracle.lmhead(h, w, row_idx=idx, inv_temperature=0.7, forbid_token=5, target=tgt_dense[idx])
    # compact outputs
    got = run_lm(h, w, row_idx=idx, inv_t=0.7, forbid=5, target=tgt_dense[idx])
    compare(got, ref)
    # dense outputs: slot row_idx[r]; untouched slots keep their fill
    got = run_lm(h, w, row_idx=idx, inv_t=0.7, forbid=5, scatter=True, target=tgt_dense)
    compare(got, ref, sel=idx)
    rest = np.setdiff1d(np.arange(R), idx)
    assert np.all(np.isnan(got["conf"][rest])) and np.all(got["tok"][rest] == -7)
    # device-side row count smaller than the host bound: only the first m rows are produced
    got = run_lm(h, w, row_idx=idx, M=41, m_dev=17, inv_t=0.7, forbid=5)
    compare({k: v[:17] for k, v in got.items()}, {k: v[:17] for k, v in ref.items() if k != "zt"})
    assert np.all(np.isnan(got["conf"][17:])) and np.all(got["tok"][17:] == -7)
    got = run_lm(h, w, row_idx=idx, M=41, m_dev=0)
    assert np.all(np.isnan(got["conf"])) and np.all(got["tok"] == -7)


@pytest.mark.parametrize("R,n_sel,variant", [(400, 300, -1), (900, 700, -1), (300, 230, 21), (300, 230, 20)])
def test_gather_mdev_target_on_the_ring_shapes(R, n_sel, variant):
    """Row gather, a device-side row count, a temperature, a forbidden token and target logits through the
    direct-to-LDS shapes the planner takes above 192 rows (two 192-row chunks, 256-row chunks, one 256-row chunk)."""
    Dh, V = 256, 1300
    h, w = rnd(31 + R, (R, Dh)), rnd(32 + R, (V, Dh), Dh ** -0.25)
    idx = np.array(sorted(np.random.default_rng(3).permutation(R)[:n_sel]), np.int32)
    tgt = np.random.default_rng(4).integers(0, V, size=n_sel).astype(np.int32)
    ref = oracle.lmhead(h, w, row_idx=idx, inv_temperature=1.3, forbid_token=777, target=tgt)
    dlm.set_option("lmhead_variant", variant)
    try:
        got = run_lm(h, w, row_idx=idx, inv_t=1.3, forbid=777, target=tgt)
        compare(got, ref)
        m = n_sel - 37
        got = run_lm(h, w, row_idx=idx, M=n_sel, m_dev=m, inv_t=1.3, forbid=777)
    finally:
        dlm.set_option("lmhead_variant", -1)
    compare({k: v[:m] for k, v in got.items()}, {k: v[:m] for k, v in ref.items() if k != "zt"})
    assert np.all(np.isnan(got["conf"][m:])) and np.all(got["tok"][m:] == -7)
    # far fewer rows on the device than the host's bound: most row tiles of the launch are dead (their wavefronts
    # only take part in the loads and barriers), down to one row and to none
    dlm.set_option("lmhead_variant", variant)
    try:
        for m in (n_sel // 2, 33, 1, 0):
            compare_prefix(run_lm(h, w, row_idx=idx, M=n_sel, m_dev=m, inv_t=1.3, forbid=777), ref, m)
    finally:
        dlm.set_option("lmhead_variant", -1)


@pytest.mark.parametrize("bound,variant", [(100, 3), (128, 3), (192, 4), (250, 5), (256, 21)])
def test_device_row_count_below_the_bound_in_row_split_shapes(bound, variant):
    """Shapes whose wavefronts split the rows run one copy of their loop per count of live row tiles."""
    Dh, V = 320, 900
    h, w = rnd(51 + bound, (bound, Dh)), rnd(52 + bound, (V, Dh), Dh ** -0.25)
    ref = oracle.lmhead(h, w, forbid_token=V - 1)
    dlm.set_option("lmhead_variant", variant)
    try:
        for m in sorted({bound, bound - 31, bound - 32, bound // 2 + 1, 65, 64, 33, 32, 1}, reverse=True):
            if m < 1 or m > bound:
                continue
            compare_prefix(run_lm(h, w, M=bound, m_dev=m, forbid=V - 1), ref, m)
    finally:
        dlm.set_option("lmhead_variant", -1)


@pytest.mark.parametrize("M", [4096, 4097])
@pytest.mark.parametrize("V,counted", [(300, 1), (300, 50), (300, -1), (33000, 1), (33000, 50)])
def test_many_rows_of_which_the_device_counts_few(M, V, counted):
    """More than 4096 rows with a device count take the reduction that looks at the count first; up to 256 partials a row (V = 300) and
    more; rows gathered and scattered, those past the count untouched."""
    m, Dh = M if counted < 0 else counted, 64
    h, w = rnd(1500 + M, (M, Dh)), rnd(1501 + V, (V, Dh), Dh ** -0.25)
    idx = np.random.default_rng(15).permutation(M).astype(np.int32)
    got = run_lm(h, w, row_idx=idx, m_dev=m, forbid=V - 1, scatter=True)
    ref = oracle.lmhead(h, w, row_idx=idx[:m], forbid_token=V - 1)
    if m >= 20:
        compare(got, ref, sel=idx[:m])
    else:
        assert np.abs(got["conf"][idx[:m]].astype(np.float64) - ref["conf"]).max() <= CONF_TOL and np.abs(got["lse"][idx[:m]] - ref["lse"]).max() <= Z_TOL
    assert np.all(np.isnan(got["conf"][idx[m:]])) and np.all(got["tok"][idx[m:]] == -7)


def test_non_temporal_w_stream_changes_nothing():
    """One row chunk: W is fetched with non-temporal loads unless the option turns that off; same bits either way."""
    h, w = rnd(71, (150, 256)), rnd(72, (3000, 256), 0.25)
    a = run_lm(h, w, forbid=11)
    dlm.set_option("lmhead_nt", 0)
    try:
        b = run_lm(h, w, forbid=11)
    finally:
        dlm.set_option("lmhead_nt", 1)
    for k in a:
        assert np.array_equal(a[k], b[k])
    with pytest.raises(dlm.DlmError):
        dlm.set_option("lmhead_nt", 2)


def test_extreme_logits_and_tiny_vocabularies():
    """Logits of magnitude ~500 (max-subtracted soft-max must not overflow), a vocabulary of one token, and one of
    two tokens with one of them forbidden (confidence exactly 1)."""
    Dh = 128
    h = synth.f32_to_bf16_bits(np.random.default_rng(1).normal(size=(70, Dh)).astype(np.float32) * 6.0)
    w = synth.f32_to_bf16_bits(np.random.default_rng(2).normal(size=(500, Dh)).astype(np.float32) * 6.0)
    ref = oracle.lmhead(h, w, forbid_token=3)
    assert np.abs(ref["zmax"]).max() > 300
    got = run_lm(h, w, forbid=3)
    assert np.all(np.isfinite(got["conf"])) and np.all(np.isfinite(got["lse"]))
    clear = (ref["zmax"] - ref["z2nd"]) >= 1e-1
    assert np.array_equal(got["tok"][clear], ref["tok"][clear])
    assert np.abs(got["conf"] - ref["conf"])[clear].max() <= 2e-2      # |logit| ~ 500 at bf16-product precision
    assert np.abs(got["lse"] - ref["lse"]).max() <= 1e-3 * np.abs(ref["lse"]).max()
    for V, forbid in ((1, -1), (2, 1), (2, 0)):
        w1 = rnd(7 + V, (V, Dh), 0.3)
        got = run_lm(rnd(8, (40, Dh)), w1, forbid=forbid)
        want_tok = 0 if forbid != 0 else 1
        assert np.all(got["tok"] == want_tok)
        if V == 1 or forbid >= 0:
            assert np.allclose(got["conf"], 1.0, atol=1e-6)
            assert np.all(got["z2nd"] == -np.inf)


def test_ties_pick_lowest_index():
    Dh, V = 64, 700
    h = synth.f32_to_bf16_bits(np.ones((40, Dh), np.float32))
    w = synth.f32_to_bf16_bits(np.full((V, Dh), 0.25, np.float32))
    got = run_lm(h, w)
    assert np.all(got["tok"] == 0)
    assert np.allclose(got["conf"], 1.0 / V, atol=1e-6)
    assert np.allclose(got["z2nd"], got["zmax"])
    got = run_lm(h, w, forbid=0)
    assert np.all(got["tok"] == 1) and np.allclose(got["conf"], 1.0 / (V - 1), atol=1e-6)
    # two equal maxima in different vocabulary tiles: the lower one wins
    wf = np.zeros((V, Dh), np.float32)
    wf[650, 0] = 2.0
    wf[131, 0] = 2.0
    got = run_lm(synth.f32_to_bf16_bits(np.eye(3, Dh, dtype=np.float32)), synth.f32_to_bf16_bits(wf))
    assert got["tok"][0] == 131 and got["z2nd"][0] == got["zmax"][0] == 2.0


@pytest.mark.parametrize("M,cus", [(20, 0), (50, 0), (90, 0), (150, 0), (250, 0), (300, 0), (520, 0), (250, 4), (300, 8), (520, 8)])
def test_logits_that_scale_to_one_value_are_a_tie(M, cus):
    """z = raw logit * inverse temperature in fp32, and the smallest token that maximises z is the answer: of two raw logits one
    unit in the last place apart that scale to the same z, the lower token wins, wherever the two lie in the vocabulary tiles."""
    Dh, V, ulp = 128, 4200, 2.0 ** -23
    t = np.float32(0.7)
    a = next(x for x in np.arange(1.0, 2.0, 2.0 ** -7, dtype=np.float32) if x * t == (x + np.float32(ulp)) * t)
    rng = np.random.default_rng(8)
    # pair j: `lo` has the raw logit a, the higher token lo + gap has a + ulp (both sums exact in fp32)
    gaps = [1, 2, 3, 4, 8, 9, 16, 24, 27, 32, 36, 64, 65, 96, 123, 128, 160, 256, 512, 1000, 2048]
    wf, lows, used = np.zeros((V, Dh), np.float32), [], set()
    for j in range(64):
        gap = gaps[j % len(gaps)]
        lo = next(v for v in rng.permutation((V - gap) // 4) * 4 if v + gap < V and not used & {v, v + gap})
        used |= {lo, lo + gap}
        wf[lo, j] = wf[lo + gap, j] = a
        wf[lo + gap, 64 + j] = 1.0
        lows.append(lo)
    pair = np.arange(M) % 64
    hf = np.zeros((M, Dh), np.float32)
    hf[np.arange(M), pair] = 1.0
    hf[np.arange(M), 64 + pair] = ulp
    dlm.set_option("lmhead_cus", cus)
    try:
        got = run_lm(synth.f32_to_bf16_bits(hf), synth.f32_to_bf16_bits(wf), inv_t=float(t))
    finally:
        dlm.set_option("lmhead_cus", 0)
    assert np.all(got["zmax"] == a * t) and np.all(got["z2nd"] == a * t)
    assert np.array_equal(got["tok"], np.asarray(lows)[pair])


def test_closed_form_threshold_boundary():
    # z = (a, 0, ..., 0): conf = e^a / (e^a + V - 1)
    Dh, V = 64, 2048
    for a in (2.0, 7.5, 9.8125):
        wf = np.zeros((V, Dh), np.float32)
        wf[1234, 0] = a
        got = run_lm(synth.f32_to_bf16_bits(np.eye(1, Dh, dtype=np.float32)), synth.f32_to_bf16_bits(wf))
        want = np.exp(a) / (np.exp(a) + V - 1)
        assert got["tok"][0] == 1234 and abs(got["conf"][0] - want) < 1e-5


def test_rerun_is_bitwise_identical():
    h, w = rnd(5, (200, 256)), rnd(6, (3000, 256), 0.25)
    a, b = run_lm(h, w), run_lm(h, w)
    for k in a:
        assert np.array_equal(a[k], b[k])


def test_full_vocabulary_sampled_rows():
    """LLaDA-8B-sized head (V = 126464, Dh = 4096), 256 rows as in the benchmark's first step;
    the oracle checks a sample of rows one by one."""
    cfg = synth.CONFIGS["c2"]
    w = synth.w_vocab(cfg)
    hid = synth.step_hidden(cfg, 0, 0).reshape(cfg.B * cfg.Lb, cfg.Dh)
    got = run_lm(hid, w, forbid=cfg.forbid_token)
    sample = np.array([0, 31, 77, 128, 200, 255], np.int32)
    ref = oracle.lmhead(hid, w, row_idx=sample, forbid_token=cfg.forbid_token)
    g = {k: v[sample] for k, v in got.items()}
    assert np.abs(g["conf"] - ref["conf"]).max() <= CONF_TOL
    clear = (ref["zmax"] - ref["z2nd"]) >= MARGIN
    assert np.array_equal(g["tok"][clear], ref["tok"][clear])
    assert np.abs(g["lse"] - ref["lse"]).max() <= 5e-3 and np.abs(g["zmax"] - ref["zmax"]).max() <= 5e-3
    # properties that hold at any size
    assert np.all(got["conf"] > 0) and np.all(got["conf"] <= 1.0 + 1e-6)
    assert np.all((got["tok"] >= 0) & (got["tok"] < cfg.V - 1))
    assert np.all(got["z2nd"] <= got["zmax"]) and np.all(got["lse"] >= got["zmax"])
    assert np.allclose(got["conf"], np.exp(got["zmax"] - got["lse"]), atol=1e-5)


@pytest.mark.parametrize("variant", [-1, 0, 3, 5, 7, 10, 16, 20, 21, 22, 25, 29])
@pytest.mark.parametrize("mode", ["margin", "neg_entropy"])
def test_alternative_confidence_scores(mode, variant):
    """conf = p(top-1) - p(top-2) or sum_v p_v log p_v instead of the token probability; every other output unchanged."""
    M, Dh, V = 300, 192, 1100
    h, w = rnd(920, (M, Dh)), rnd(921, (V, Dh), Dh ** -0.25)
    ref = oracle.lmhead(h, w, forbid_token=V - 1, inv_temperature=0.8)
    hd, wd = bf16_dev(h), bf16_dev(w)
    cm = dlm.CONF_MARGIN if mode == "margin" else dlm.CONF_NEG_ENTROPY
    conf = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
    tok = torch.full((M,), -7, dtype=torch.int32, device=DEV)
    ws = torch.empty(dlm.lmhead_workspace_bytes(M, V, conf_mode=cm), dtype=torch.uint8, device=DEV)
    dlm.set_option("lmhead_variant", variant)
    try:
        dlm.lmhead_confidence(hd, wd, conf, tok, forbid_token=V - 1, inv_temperature=0.8, lse=lse, workspace=ws, conf_mode=cm)
        torch.cuda.synchronize()
    finally:
        dlm.set_option("lmhead_variant", -1)
    got = conf.cpu().numpy().astype(np.float64)
    tol = CONF_TOL if mode == "margin" else Z_TOL          # the entropy lives on the logits' scale
    assert np.abs(got - ref[mode]).max() <= tol
    clear = (ref["zmax"] - ref["z2nd"]) >= MARGIN
    assert np.array_equal(tok.cpu().numpy()[clear], ref["tok"][clear])
    assert np.abs(lse.cpu().numpy() - ref["lse"]).max() <= Z_TOL
    if mode == "neg_entropy":
        assert np.all(got <= 1e-4) and np.all(got >= -np.log(V) - 1e-3)


def test_entropy_full_vocabulary_and_sampling_together():
    """LLaDA-sized head: negative entropy on sampled rows; with sampling on, the score is that of the distribution
    while the token is the drawn one."""
    from oracle import sampling
    cfg = synth.CONFIGS["c2"]
    w = synth.w_vocab(cfg)
    hid = synth.step_hidden(cfg, 0, 1).reshape(-1, cfg.Dh)
    idx = np.sort(np.random.default_rng(5).permutation(hid.shape[0])[:70]).astype(np.int32)
    M = len(idx)
    conf = torch.zeros(M, dtype=torch.float32, device=DEV)
    tok = torch.zeros(M, dtype=torch.int32, device=DEV)
    ws = torch.empty(dlm.lmhead_workspace_bytes(M, cfg.V, sample=True, conf_mode=dlm.CONF_NEG_ENTROPY), dtype=torch.uint8, device=DEV)
    dlm.lmhead_confidence(bf16_dev(hid), bf16_dev(w), conf, tok, M=M, row_idx=dev(idx), forbid_token=cfg.forbid_token,
                          workspace=ws, conf_mode=dlm.CONF_NEG_ENTROPY, sample_seed=99, sample_step=4)
    torch.cuda.synchronize()
    pick = np.array([0, 13, 41, 69])
    ref = oracle.lmhead(hid, w, row_idx=idx[pick], forbid_token=cfg.forbid_token)
    smp = sampling.lmhead_sampled(hid, w, seed=99, step=4, row_idx=idx[pick], forbid_token=cfg.forbid_token)
    assert np.abs(conf.cpu().numpy()[pick] - ref["neg_entropy"]).max() <= Z_TOL
    clear = (smp["pmax"] - smp["p2nd"]) >= MARGIN
    assert np.array_equal(tok.cpu().numpy()[pick][clear], smp["tok"][clear])


@pytest.mark.parametrize("M,m_dev,guess", [(256, 120, 125), (256, 130, 125), (256, 128, 128), (256, 129, 100), (200, 40, 60),
                                           (200, 65, 60), (100, 20, 30), (100, 33, 30), (64, 10, 20), (500, 200, 250),
                                           (500, 300, 250), (500, 500, 250), (300, 0, 100), (128, 128, 90), (70, 70, 1)])
def test_expected_row_count_only_selects_the_shape(M, m_dev, guess):
    """M_expected queues the shape for the guessed count, guarded by the device's count, in front of the shape for the
    bound: whether the guess holds (count within that shape's capacity) or not, the outputs are the oracle's and,
    up to the rounding of another summation order, those of a call without a guess."""
    Dh, V = 256, 1500
    h, w = rnd(7100 + M, (M, Dh)), rnd(7200 + M, (V, Dh), Dh ** -0.25)
    idx = np.arange(M - 1, -1, -1).astype(np.int32)            # gathered rows, reversed
    plain = run_lm(h, w, row_idx=idx, M=M, m_dev=m_dev, forbid=V - 1)
    guessed = run_lm(h, w, row_idx=idx, M=M, m_dev=m_dev, forbid=V - 1, M_expected=guess)
    assert np.array_equal(np.isnan(plain["conf"]), np.isnan(guessed["conf"]))
    assert np.allclose(plain["conf"][:m_dev], guessed["conf"][:m_dev], rtol=0, atol=2e-6)
    assert np.allclose(plain["lse"][:m_dev], guessed["lse"][:m_dev], rtol=0, atol=1e-4)
    assert np.array_equal(plain["tok"], guessed["tok"])
    ref = oracle.lmhead(h, w, row_idx=idx[:m_dev], forbid_token=V - 1)
    compare_prefix(guessed, ref, m_dev)


def test_expected_row_count_with_sampling_and_entropy_partials():
    """The second partial array sits at another offset in the guessed shape's layout: sampled tokens and the
    entropy confidence must not depend on the guess either (beyond rounding)."""
    M, Dh, V = 200, 256, 3000
    h, w = bf16_dev(rnd(7301, (M, Dh))), bf16_dev(rnd(7302, (V, Dh), Dh ** -0.25))
    for kw in (dict(sample_seed=11, sample_step=3), dict(conf_mode=dlm.CONF_NEG_ENTROPY)):
        outs = []
        for guess, md in ((0, 50), (60, 50), (60, 70)):
            conf = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
            tok = torch.full((M,), -7, dtype=torch.int32, device=DEV)
            ws = torch.empty(dlm.lmhead_workspace_bytes(M, V, sample="sample_seed" in kw, conf_mode=kw.get("conf_mode", dlm.CONF_TOKEN_PROB)),
                             dtype=torch.uint8, device=DEV)
            dlm.lmhead_confidence(h, w, conf, tok, M=M, m_dev=dev(np.asarray([md], np.int32)), workspace=ws,
                                  M_expected=guess, **kw)
            torch.cuda.synchronize()
            outs.append((conf.cpu().numpy(), tok.cpu().numpy()))
        # the same tokens; confidences up to the rounding of another summation order
        assert np.array_equal(outs[0][1], outs[1][1]) and np.array_equal(outs[0][1][:50], outs[2][1][:50])
        assert np.allclose(outs[0][0], outs[1][0], rtol=0, atol=1e-5, equal_nan=True)
        assert np.allclose(outs[0][0][:50], outs[2][0][:50], rtol=0, atol=1e-5)
        assert not np.isnan(outs[2][0][:70]).any() and np.isnan(outs[2][0][70:]).all()


@pytest.mark.parametrize("M,cus,V", [(70, 8, 2600), (100, 8, 2400), (128, 4, 1500), (150, 8, 2561), (192, 8, 2300), (230, 8, 2500),
                                     (256, 6, 2047), (96, 8, 2305)])
def test_half_height_tail_launch(M, cus, V):
    """A vocabulary whose tile count leaves the last round of workgroups at most half full is covered by full-height tiles and, in the
    same launch, half-height ones for the tail.  The assumed CU count is lowered so that a small problem
    takes that path (e.g. 2600 rows = 11 tiles of 256 on 8 'CUs': 8 full tiles + 5 half tiles, the last one ragged);
    every output against the oracle, with a forbidden token in the tail and targets on both sides of the seam."""
    Dh = 128
    h, w = rnd(1300 + M, (M, Dh)), rnd(1301 + M, (V, Dh), Dh ** -0.25)
    tgt = np.random.default_rng(M).integers(0, V, size=M).astype(np.int32)
    tgt[:4] = [0, V - 2, (V // 256 // cus * cus) * 256 - 1, min(V - 2, (V // 256 // cus * cus) * 256)]   # around the seam
    ref = oracle.lmhead(h, w, forbid_token=V - 1, target=tgt)
    dlm.set_option("lmhead_cus", cus)
    try:
        got = run_lm(h, w, forbid=V - 1, target=tgt)
        compare(got, ref)
        # device-side row count below the bound, and two queued shapes on top of the tail
        m_dev = max(1, M - 37)
        got = run_lm(h, w, forbid=V - 1, m_dev=m_dev, M_expected=max(1, int(0.8 * M)))
        compare_prefix(got, ref, m_dev)
    finally:
        dlm.set_option("lmhead_cus", 0)
    # and with the tail rule switched off the same values up to summation order
    dlm.set_option("lmhead_cus", -1)
    try:
        compare(run_lm(h, w, forbid=V - 1, target=tgt), ref)
    finally:
        dlm.set_option("lmhead_cus", 0)


@pytest.mark.parametrize("M,m_dev,Dh,V,cus", [
    (257, None, 128, 2100, 8),      # shape of 192-row chunks, the shortest walk a queue takes, more lists than CUs
    (960, 300, 192, 1100, 8),       # two of four chunks counted; 5 vocabulary tiles: three of the eight lists are empty
    (384, 192, 128, 4000, 16),      # the device counts one chunk less than the bound
    (470, None, 256, 2817, 8),      # 256-row chunks, a last vocabulary tile of one token
    (580, 300, 128, 3000, 16),
    (580, 256, 192, 3000, 8),
    (700, 0, 128, 3000, 8),         # nothing counted
    (700, 1, 128, 3000, 8),
    (1700, 1400, 128, 2500, 8),     # seven chunks (blocks of seven), six of them counted
    (2049, None, 128, 2600, 16),    # nine chunks, one row in the last; the last group of vocabulary tiles incomplete
])
def test_workgroups_that_take_their_tiles_from_a_queue(M, m_dev, Dh, V, cus):
    """More tiles than workgroups, against the oracle, and (all rows counted) bit for bit what one workgroup a tile gives.  The shape is the one for
    the row count by name: without the lowered CU count such small vocabularies take smaller tiles, which sum in another order."""
    R = M + 50
    h, w = rnd(940 + M, (R, Dh)), rnd(941 + V, (V, Dh), Dh ** -0.25)
    idx = np.random.default_rng(M).permutation(R)[:M].astype(np.int32)
    kw = dict(row_idx=idx, M=M, m_dev=m_dev, forbid=V - 1, inv_t=0.9)
    m = M if m_dev is None else m_dev
    ref = oracle.lmhead(h, w, row_idx=idx[:m], forbid_token=V - 1, inv_temperature=0.9) if m else None
    dlm.set_option("lmhead_variant", 22 if M <= 384 else 20)
    try:
        plain = run_lm(h, w, **kw)
        dlm.set_option("lmhead_cus", cus)
        queued = [run_lm(h, w, **kw) for _ in range(2)]
    finally:
        dlm.set_option("lmhead_cus", 0)
        dlm.set_option("lmhead_variant", -1)
    for got in queued:
        compare_prefix(got, ref, m)
        if m_dev is None:
            assert all(np.array_equal(got[k], plain[k], equal_nan=True) for k in plain)


@pytest.mark.parametrize("m_dev", [None, 900, 600])
def test_every_value_of_the_blocking_option(m_dev):
    """Blocks of workgroups per XCD change the order of the tiles and where a tile's walk over Dh starts, and the values >= 0 also
    switch the queue off.  The device's count leaves every chunk, all but one and half of them.  Against the oracle: 128 products summed in
    fp32 in any order stay within 128 * 2^-24 * sum |h w| < 128 * 2^-24 * 128 = 1e-3 of the exact sum, below Z_TOL."""
    h, w = rnd(1700, (1100, 128)), rnd(1701, (3000, 128), 128 ** -0.25)
    ref = oracle.lmhead(h[:m_dev], w, forbid_token=7)
    dlm.set_option("lmhead_cus", 8)
    try:
        for block in (-1, 0, 1, 4, 8):
            dlm.set_option("lmhead_block", block)
            compare_prefix(run_lm(h, w, m_dev=m_dev, forbid=7), ref, m_dev or 1100)
    finally:
        dlm.set_option("lmhead_block", -1)
        dlm.set_option("lmhead_cus", 0)


@pytest.mark.parametrize("kind", ["plain", "static", "strided", "margin", "entropy", "sampled", "sampled_entropy", "target_scatter"])
@pytest.mark.parametrize("M,Dh,V,cus,counted", [
    (300, 128, 2100, 8, (300,)),                        # 192-row chunks, the shortest walk a queue takes
    (580, 192, 2817, 8, (580, 300)),                    # 256-row chunks, all counted and two of three; a last vocabulary tile of one token
    (580, 128, 3000, 16, (200, 385, 384)),              # guess 300: both shapes queued for the call have a queue, the first runs, then the second
    (580, 128, 3000, 8, (100, 140)),                    # guess 100: the one-chunk shape clears the counters of the other
])
def test_every_form_of_a_call_through_a_queue(kind, M, Dh, V, cus, counted):
    """The forms that the tiles of a queue take their own way: the noise's kernel, the second partials (behind which the counters lie) and
    the runner-up in the free stage of the ring, targets stored between two tiles, other strides, the library's own scratch, two
    queued shapes.  The counters start with what the workspace held: 0x5A bytes at first, then what the last call left."""
    from oracle import sampling
    guess = {200: 300, 385: 300, 384: 300, 100: 100, 140: 100}.get(counted[0], 0)
    R = M + 37
    h, w = rnd(1800 + M, (R, Dh)), rnd(1801 + V, (V, Dh), Dh ** -0.25)
    idx = np.random.default_rng(M).permutation(R)[:M].astype(np.int32)
    pad = 24 if kind == "strided" else 0
    hd, wd = torch.zeros((R, Dh + pad), dtype=torch.bfloat16, device=DEV), torch.zeros((V, Dh + 2 * pad), dtype=torch.bfloat16, device=DEV)
    hd[:, :Dh], wd[:, :Dh] = bf16_dev(h), bf16_dev(w)
    sample, ent, scatter = "sampled" in kind, "entropy" in kind, kind == "target_scatter"
    mode = dlm.CONF_NEG_ENTROPY if ent else dlm.CONF_MARGIN if kind == "margin" else dlm.CONF_TOKEN_PROB
    tgt = np.random.default_rng(V).integers(0, V - 1, size=R).astype(np.int32)
    ref = oracle.lmhead(h, w, row_idx=idx, forbid_token=V - 1, inv_temperature=0.8, target=tgt[idx])
    smp = sampling.lmhead_sampled(h, w, seed=77, step=5, stream=2, row_idx=idx, forbid_token=V - 1, inv_temperature=0.8) if sample else None
    want = smp["conf"] if sample and not ent else ref["neg_entropy"] if ent else ref["margin"] if kind == "margin" else ref["conf"]
    top, second = (smp["pmax"], smp["p2nd"]) if sample else (ref["zmax"], ref["z2nd"])
    want_tok = smp["tok"] if sample else ref["tok"]
    gw = GuardedWorkspace(dlm.lmhead_workspace_bytes(M, V, sample=sample, conf_mode=mode))
    gw.ws.fill_(0x5A)
    n_out = R if scatter else M
    dlm.set_option("lmhead_cus", cus)
    try:
        for m in counted:
            f = lambda: torch.full((n_out,), float("nan"), dtype=torch.float32, device=DEV)
            conf, lse, zt, tok = f(), f(), f(), torch.full((n_out,), -7, dtype=torch.int32, device=DEV)
            kw = dict(M=M, row_idx=dev(idx), m_dev=None if m == M else dev(np.asarray([m], np.int32)), M_expected=guess, forbid_token=V - 1,
                      inv_temperature=0.8, lse=lse, conf_mode=mode, out_scatter=scatter)
            if sample:
                kw.update(sample_seed=77, sample_step=5, sample_stream=2)
            if scatter:
                kw.update(target=dev(tgt), ztarget=zt)
            kw.update(static_scratch=True) if kind == "static" else kw.update(workspace=gw.ws)
            dlm.lmhead_confidence(hd[:, :Dh], wd[:, :Dh], conf, tok, **kw)
            gw.check()
            at = idx[:m] if scatter else np.arange(m)
            conf, lse, zt, tok = conf.cpu().numpy(), lse.cpu().numpy(), zt.cpu().numpy(), tok.cpu().numpy()
            clear = (top - second)[:m] >= MARGIN
            assert clear.mean() > 0.9 and np.array_equal(tok[at][clear], want_tok[:m][clear])
            same = tok[at] == want_tok[:m] if sample and not ent else np.ones(m, bool)
            assert np.abs(conf[at][same].astype(np.float64) - want[:m][same]).max() <= (Z_TOL if ent else CONF_TOL)
            assert np.abs(lse[at] - ref["lse"][:m]).max() <= Z_TOL
            if scatter:
                assert np.abs(zt[at] - ref["zt"][:m]).max() <= Z_TOL
            rest = np.setdiff1d(np.arange(n_out), at)
            assert np.all(np.isnan(conf[rest])) and np.all(tok[rest] == -7) and np.all(np.isnan(zt[rest]))
    finally:
        dlm.set_option("lmhead_cus", 0)


@pytest.mark.parametrize("M,m_dev,Dh,V,guess", [
    (33, None, 64, 100, 0), (64, 40, 64, 129, 0),          # 128 x 32 tiles instead of 128 x 64, the shortest walk
    (65, None, 320, 2100, 0), (256, 97, 512, 4096, 120),   # 128 x 32, all 256 of them; a count with whole chunks past it
    (256, 255, 512, 4097, 200), (200, None, 128, 5000, 0), # one vocabulary tile more: 128 x 64
    (384, None, 512, 10000, 0), (385, 129, 576, 2200, 0),  # 128 x 128 and 128 x 32
    (500, 3, 512, 17000, 0), (1030, None, 512, 300, 0),    # 256 x 128; more row chunks than vocabulary tiles
    (256, 200, 64, 40960, 0), (256, 200, 64, 40961, 0),    # 160 tiles of 256 x 256, the most that are few, and one more
    (256, 90, 64, 40960, 100), (256, 110, 4096, 33000, 120), (256, 200, 4096, 33000, 120),   # the bound's shape stays the large one: a guess that is not
    (512, 100, 512, 17000, 120), (1024, 200, 1024, 5000, 80),                                # worth it, one that is, right and wrong
    (1405, None, 64, 3887, 0), (1059, 700, 128, 4701, 0), (700, 650, 64, 10000, 0),          # blocks of 2, 3 and 5 vocabulary tiles an XCD
])
def test_small_vocabularies_take_small_tiles(M, m_dev, Dh, V, guess):
    """The shapes that fill the chip where the one for the row count alone leaves most of it idle, on both sides of the lines between them."""
    R = M + 19
    h, w = rnd(1900 + M, (R, Dh)), rnd(1901 + V, (V, Dh), Dh ** -0.25)
    idx = np.random.default_rng(M + V).permutation(R)[:M].astype(np.int32)
    m = m_dev or M
    ref = oracle.lmhead(h, w, row_idx=idx[:m], forbid_token=V - 1, inv_temperature=0.9)
    compare_prefix(run_lm(h, w, row_idx=idx, M=M, m_dev=m_dev, inv_t=0.9, forbid=V - 1, M_expected=guess), ref, m)


@pytest.mark.parametrize("R,n_sel,variant", [(400, 300, 22), (900, 700, 20)])
def test_gather_on_the_ring_shapes_by_name(R, n_sel, variant):
    test_gather_mdev_target_on_the_ring_shapes(R, n_sel, variant)


def test_expected_row_counts_where_tiles_are_many():
    dlm.set_option("lmhead_cus", 8)
    try:
        for M, m_dev, guess in ((256, 150, 160), (256, 200, 160), (500, 200, 250), (500, 300, 250), (300, 0, 100), (100, 33, 30)):
            test_expected_row_count_only_selects_the_shape(M, m_dev, guess)
        test_expected_row_count_with_sampling_and_entropy_partials()
    finally:
        dlm.set_option("lmhead_cus", 0)


@pytest.mark.parametrize("M,expected,counted,V,Dh", [
    (1024, 81, 76, 5000, 4096), (512, 128, 121, 16000, 4096), (384, 96, 91, 16000, 4096), (256, 128, 121, 20000, 4096),   # the bound's tiles: 256 x 128
    (1024, 250, 243, 10000, 1024), (1024, 81, 76, 10000, 1024), (512, 40, 38, 20000, 1024),                               # 256 x 256
])
def test_a_right_guess_runs_the_shape_of_its_own_rows(M, expected, counted, V, Dh):
    """Small vocabularies, where the bound alone would leave most CUs without a row that counts: the outputs are, bit for bit, those of a call
    whose bound is the guessed shape's capacity (the shapes group the vocabulary differently, so another shape rounds its sums otherwise)."""
    g = torch.Generator(device=DEV).manual_seed(M + V)
    h = torch.randn(M, Dh, generator=g, device=DEV, dtype=torch.bfloat16)
    w = torch.randn(V, Dh, generator=g, device=DEV, dtype=torch.bfloat16) * Dh ** -0.25
    cap = next(c for c in (32, 64, 128, 192, 256, 384) if expected <= c)
    outs = []
    for bound, guess in ((M, expected), (cap, 0)):
        conf, lse = (torch.full((M,), float("nan"), device=DEV) for _ in range(2))
        tok = torch.full((M,), -7, dtype=torch.int32, device=DEV)
        ws = torch.empty(dlm.lmhead_workspace_bytes(bound, V), dtype=torch.uint8, device=DEV)
        dlm.lmhead_confidence(h, w, conf, tok, M=bound, m_dev=dev(np.asarray([counted], np.int32)), forbid_token=V - 1, lse=lse, workspace=ws,
                              M_expected=guess)
        outs.append((conf, lse, tok))
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert not outs[0][0][:counted].isnan().any() and outs[0][0][counted:].isnan().all()


@pytest.mark.parametrize("M,Dh,V,shape", [(257, 64, 300, 0), (300, 448, 20000, 3), (512, 256, 4096, 29), (700, 192, 3000, 25), (4096, 128, 2048, 3),
                                          (1503, 64, 5318, 20), (372, 64, 2365, 29), (716, 64, 2383, 25)])   # 36 of a smaller tile on an XCD
def test_small_tiles_whatever_the_hidden_size(M, Dh, V, shape):
    """More than 256 rows of fewer than 512 elements: the shape that fills the chip, bit for bit as by name, and the oracle's values."""
    h, w = rnd(2000 + M, (M, Dh)), rnd(2001 + V, (V, Dh), Dh ** -0.25)
    got = run_lm(h, w, forbid=V - 1)
    dlm.set_option("lmhead_variant", shape)
    try:
        named = run_lm(h, w, forbid=V - 1)
    finally:
        dlm.set_option("lmhead_variant", -1)
    assert all(np.array_equal(got[k], named[k], equal_nan=True) for k in named)
    compare(got, oracle.lmhead(h, w, forbid_token=V - 1))


@pytest.mark.parametrize("kind", ["plain", "static", "strided", "margin", "entropy", "sampled", "sampled_entropy", "target_scatter"])
@pytest.mark.parametrize("M,Dh,V,counted", [(90, 128, 2049, (90, 33)), (512, 256, 4096, (512, 300)), (700, 192, 3000, (700, 40))])
def test_every_form_of_a_call_of_a_small_vocabulary(kind, M, Dh, V, counted):
    """Tiles of 128 x 32, 128 x 64 and 128 x 128, all rows counted and with whole chunks past the count."""
    test_every_form_of_a_call_through_a_queue(kind, M, Dh, V, 0, counted)


@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("counted", [90, 2200])
def test_a_guess_of_narrow_tiles_leaves_the_bound_its_queue(counted, sample):
    """The guess's tiles of 128 tokens make as many partials a row as the workspace has room for, but of its own rows alone: the counters of the
    bound's queue (one in each of the last eight lines) still fit behind them.  Either launch gives what its shape gives without the other."""
    M, Dh, V, expected = 2300, 128, 16000, 100
    g = torch.Generator(device=DEV).manual_seed(71)
    h = torch.randn(M, Dh, generator=g, device=DEV, dtype=torch.bfloat16)
    w = torch.randn(V, Dh, generator=g, device=DEV, dtype=torch.bfloat16) * Dh ** -0.25
    ws = torch.full((dlm.lmhead_workspace_bytes(M, V, sample=sample),), 0xFF, dtype=torch.uint8, device=DEV)
    outs = []
    for bound, guess in ((M, expected), (M, 0) if counted > 128 else (128, 0)):
        conf, lse = (torch.full((M,), float("nan"), device=DEV) for _ in range(2))
        tok = torch.full((M,), -7, dtype=torch.int32, device=DEV)
        dlm.lmhead_confidence(h, w, conf, tok, M=bound, m_dev=dev(np.asarray([counted], np.int32)), lse=lse, workspace=ws, M_expected=guess,
                              **(dict(sample_seed=5, sample_step=1) if sample else {}))
        if guess:
            drawn = ws[-512:].view(torch.int32)[::16].cpu()
            assert (drawn >= 0).all() and (counted <= 128 or (drawn > 0).all()), drawn
        outs.append((conf, lse, tok))
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert not outs[0][0][:counted].isnan().any() and outs[0][0][counted:].isnan().all()
