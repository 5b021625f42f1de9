"""The library's calls under HIP graph capture (GPU): they only launch kernels on the caller's stream (no allocation, no
memset, no synchronisation), so a captured step can be replayed; dlm_lmhead_confidence_static exists for exactly such callers.
Every replay is compared with an eager call on the same inputs, with eager work between the replays."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2604_04215_amd import binding as dlm
from gpu_util import DEV, bf16_dev, rnd

pytestmark = pytest.mark.gpu


def test_attention_and_static_lm_head_replayed_from_a_graph():
    B, Lq, Hq, Hkv, d, P = 2, 32, 8, 2, 128, 300
    M, V, Dh = B * Lq, 3000, 256
    q = bf16_dev(rnd(50, (B, Lq, Hq, d)))
    ck, cv = bf16_dev(rnd(51, (B, Hkv, P, d))), bf16_dev(rnd(52, (B, Hkv, P, d)))
    kb, vb = bf16_dev(rnd(53, (B, Hkv, Lq, d))), bf16_dev(rnd(54, (B, Hkv, Lq, d)))
    out = torch.zeros_like(q)
    h = bf16_dev(rnd(55, (M, Dh)))
    w = bf16_dev(rnd(56, (V, Dh), std=Dh ** -0.25))
    conf = torch.zeros(M, device=DEV)
    tok = torch.zeros(M, dtype=torch.int32, device=DEV)

    def step():
        dlm.block_attn(q, out, prefix=(ck, cv, 0), block=(kb, vb, P), suffix=None, mask_mode=dlm.MASK_FULL)
        dlm.lmhead_confidence(h, w, conf, tok, forbid_token=V - 1, static_scratch=True)

    step()                                   # eager first: the first call on a device looks up the scratch address
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        step()                               # the binding passes torch's current stream: the capturing one
    for rep in range(3):
        q.copy_(bf16_dev(rnd(60 + rep, (B, Lq, Hq, d))))          # eager work between replays: new inputs in place
        h.copy_(bf16_dev(rnd(70 + rep, (M, Dh))))
        out.zero_(); conf.fill_(-1.0); tok.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (out, conf, tok)]
        out.zero_(); conf.fill_(-1.0); tok.fill_(-1)
        step()
        torch.cuda.synchronize()
        for a, b in zip(got, (out, conf, tok)):
            assert torch.equal(a, b), f"replay {rep} differs from the eager call"
        assert float(conf.min()) > 0 and int(tok.min()) >= 0


@pytest.mark.parametrize("M,guess,launches", [(700, 0, 3), (580, 300, 4), (580, 100, 3)])
def test_lm_head_with_a_queue_of_tiles_replayed_from_a_graph(M, guess, launches):
    """The counters that hand out the tiles are cleared inside the captured call: every replay finds them as the one before it left
    them.  With a guess two shapes are captured and the device's count, changed between replays, says which runs.  The first launch
    of a call clears the counters; it is one for that alone only where it would use them itself."""
    V, Dh = 3000, 128
    h = bf16_dev(rnd(80, (M, Dh)))
    w = bf16_dev(rnd(81, (V, Dh), std=Dh ** -0.25))
    md = torch.full((1,), M, dtype=torch.int32, device=DEV)
    conf, tok = torch.zeros(M, device=DEV), torch.zeros(M, dtype=torch.int32, device=DEV)
    step = lambda: dlm.lmhead_confidence(h, w, conf, tok, m_dev=md, M_expected=guess, forbid_token=V - 1, static_scratch=True)
    dlm.set_option("lmhead_cus", 8)
    try:
        step()
        torch.cuda.synchronize()
        graph, side = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=side):
            step()
        n = C.c_size_t()
        assert dlm.lib().hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(n)) == 0 and n.value == launches
        for rep, count in enumerate((M, 90, 350, M, 200, 90)):
            h.copy_(bf16_dev(rnd(90 + rep, (M, Dh))))
            md.fill_(count)
            conf.fill_(-1.0); tok.fill_(-1)
            graph.replay()
            torch.cuda.synchronize()
            got = conf.clone(), tok.clone()
            conf.fill_(-1.0); tok.fill_(-1)
            step()
            torch.cuda.synchronize()
            assert torch.equal(got[0], conf) and torch.equal(got[1], tok), f"replay {rep} differs from the eager call"
            assert float(conf[:count].min()) > 0 and bool((conf[count:] == -1).all())
    finally:
        dlm.set_option("lmhead_cus", 0)
