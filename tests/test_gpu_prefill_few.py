"""Chunks of few tokens, which take one pass over keys and values: edges of its groups of 32 tokens and rows, of its 128-slot
tiles (half of the last one outside the memory) and of the range it is chosen for, against the oracle."""
import numpy as np
import pytest

import bct_synth as syn
from _util import f64, make_pair, to_dev, to_np
from test_gpu_gate import gdev, gates
from test_gpu_prefill import PF_WEIGHT_REL, check_prefill_out, check_prefill_state, prefill_mass
from _util import bf16_ulp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2411_15785_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def R():
    from oracle import bct_ref
    return bct_ref


# one tile of slots (the output is finished in the pass), two, several; 1, 31, 32, 33 tokens; rows up to 32, 33 to 64 and beyond
CASES = [(1, 1, 1, 64, 1, 0), (2, 3, 1, 64, 31, 0), (1, 2, 1, 128, 32, 1), (3, 2, 1, 192, 33, 0), (1, 3, 2, 192, 16, 1),
         (2, 1, 3, 320, 11, 0), (1, 2, 8, 1088, 4, 0), (1, 1, 8, 128, 5, 1), (2, 2, 4, 64, 16, 0), (1, 1, 1, 2112, 55, 0),
         (1, 2, 1, 128, 64, 0), (1, 1, 1, 1088, 64, 0), (1, 1, 1, 1088, 54, 0), (1, 2, 5, 256, 12, 0), (3, 1, 5, 448, 13, 1), (17, 4, 1, 192, 40, 0), (16, 4, 1, 192, 40, 0),
         (16, 4, 1, 320, 40, 0), (17, 4, 1, 320, 40, 0)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hkv,G,M,T,seq", CASES)
def test_chunk(P, R, d, B, Hkv, G, M, T, seq):
    w = syn.Workload("few", 1, B, Hkv * G, Hkv, d, M, "bf16", 0)
    # a cache sized for longer chunks as well: the scratch is where that one's is
    ref, gpu, mk, mv, _ = make_pair(w, R.RefCache, P.BctCache, flags=seq, mv0=True, max_prefill_T=T + 130 * (M == 192))
    # beyond the border: too many rows, too many for the scratch, too many memories of several tiles
    several = (B, M, T) in ((3, 448, 13), (3, 192, 33), (1, 1088, 64), (17, 192, 40), (16, 192, 40), (17, 320, 40))
    assert P.bct_plan_prefill(gpu.desc, T) == (P.BCT_OK, 0 if several else 1)
    for chunk in range(2):
        q, wq, wv = syn.make_step(w, chunk * T, T=T)
        before = ref.values()
        gpu.set_values(to_dev(before, "bf16"))
        o_ref = ref.prefill(q, wq, wv, T)
        o = gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T)
        what = f"d={d} G={G} M={M} T={T} chunk {chunk}"
        check_prefill_out(to_np(o, "bf16"), o_ref, "bf16", what)
        check_prefill_state(R, ref, mk, wq, wv, to_np(gpu.values_view(), "bf16"), T, what)
    assert np.array_equal(to_np(gpu.keys_view(), "bf16"), mk)


@pytest.mark.parametrize("rs,ws", [(-0.08, 0.09), (0.09, -0.12), (0.0, 0.09)])
def test_step_sizes_and_scales(P, R, rs, ws):
    """Step sizes of either sign and zero, scales of either sign: every token's weight and every row's order turned round."""
    B, Hkv, G, d, M, T = 2, 2, 2, 128, 320, 15
    w = syn.Workload("few_gate", 1, B, Hkv * G, Hkv, d, M, "bf16", 0)
    ref, gpu, mk, mv, _ = make_pair(w, R.RefCache, P.BctCache, read_scale=rs, write_scale=ws, mv0=True, max_prefill_T=T)
    assert P.bct_plan_prefill(gpu.desc, T) == (P.BCT_OK, 1)
    q, wq, wv = syn.make_step(w, 0, T=T)
    g = gates(5, (B, T, Hkv))
    g[:, ::3] *= -1.0
    g[:, 1] = 0.0
    o_ref = ref.prefill(q, wq, wv, T, gate=g)
    o = gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T, gate=gdev(g))
    check_prefill_out(to_np(o, "bf16"), o_ref, "bf16", "gated")
    aux = R.RefCache(M, B, Hkv * G, Hkv, d, "bf16", rs, ws, 0)
    aux.set_keys(mk)
    aux.prefill(None, wq, syn.pack(np.ones(wv.shape), "bf16"), T, gate=np.abs(g))
    bound = f64(aux.values(), "bf16")[..., :1] * np.max(np.abs(f64(wv, "bf16")), axis=1)[..., None, :] * 1.01
    r = f64(ref.values(), "bf16")
    dlt = np.abs(f64(to_np(gpu.values_view(), "bf16"), "bf16") - r)
    assert np.all(dlt <= bf16_ulp(r) * 1.0001 + PF_WEIGHT_REL * bound)


def test_repeats_itself_and_replays(P):
    """Equal bits twice, and from a graph whose scratch another chunk has used in between."""
    import torch
    w = syn.Workload("few_bits", 1, 3, 8, 4, 128, 320, "bf16", 0)
    c = [P.BctCache(w.M, w.B, w.Hq, w.Hkv, w.d, torch.bfloat16, w.scale, w.scale, max_prefill_T=64) for _ in range(2)]
    ins = [to_dev(a, "bf16") for a in syn.make_step(w, 0, T=9)]
    long = [to_dev(a, "bf16") for a in syn.make_step(w, 1, T=64)]
    o = [torch.empty_like(ins[0]) for _ in range(2)]
    for x in c:
        x.set_keys(to_dev(syn.make_keys(w), "bf16"))
    c[1].prefill(*ins, 9, o[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c[1].prefill(*ins, 9, o[1])
    for x in c:
        x.set_values(None)
    for _ in range(3):
        c[0].prefill(*ins, 9, o[0])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o[0].view(torch.int16), o[1].view(torch.int16))
        assert torch.equal(c[0].values_view().view(torch.int16), c[1].values_view().view(torch.int16))
        for x in c:
            x.prefill(*long, 64)


@pytest.mark.parametrize("d,G,T,first", [(64, 1, 5, 128), (128, 1, 5, 0), (128, 4, 12, 128), (64, 2, 24, 192)])
def test_slots_masked_by_their_keys(P, R, d, G, T, first):
    """Keys whose scores overflow to -inf take no weight, also where they are all of a 128-slot tile."""
    B, Hkv, M = 2, 2, 320
    w = syn.Workload("few_masked", 1, B, Hkv * G, Hkv, d, M, "bf16", 0)
    ref, gpu, mk, mv, _ = make_pair(w, R.RefCache, P.BctCache, mv0=True, max_prefill_T=T)
    assert P.bct_plan_prefill(gpu.desc, T) == (P.BCT_OK, 1)
    keys = f64(mk, "bf16")
    keys[:, first:first + 128] = 0.0
    keys[:, first:first + 128, 0] = -3e38
    mk = syn.pack(keys, "bf16")
    gpu.set_keys(to_dev(mk, "bf16"))
    ref.set_keys(mk)
    q, wq, wv = (f64(a, "bf16") for a in syn.make_step(w, 0, T=T))
    q[..., 0] = wq[..., 0] = 2.0
    q, wq, wv = (syn.pack(a, "bf16") for a in (q, wq, wv))
    o_ref = ref.prefill(q, wq, wv, T)
    o = gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T)
    check_prefill_out(to_np(o, "bf16"), o_ref, "bf16", "masked")
    got = to_np(gpu.values_view(), "bf16")
    check_prefill_state(R, ref, mk, wq, wv, got, T, "masked")
    assert np.array_equal(got[:, :, first:first + 128], mv[:, :, first:first + 128])
