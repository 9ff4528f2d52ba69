"""The decode step that takes whole memories through one launch: where it is chosen, at the edges of its tiles and
loads, against the oracle and against the streaming launches of the same step."""
import numpy as np
import pytest

import bct_synth as syn
from _util import bf16_ulp, f64, make_pair, to_dev, to_np
from test_gpu_parity import check_out, check_state_one_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2411_15785_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def R():
    from oracle import bct_ref
    return bct_ref


# B, Hq, Hkv, d, M, dtype, per-sequence keys, workgroups per memory, threads.  A tile of keys is 16 slots for each of 8 or 16
# wavefronts (M / 16 tiles: one, two, three and more rounds, the last one partial), a lane has 4, 8 or 16 loads.
CASES = [
    (1, 1, 1, 128, 64, "bf16", 0, 2, 512),       # 4 tiles for 8 wavefronts, one memory
    (3, 5, 5, 128, 192, "bf16", 0, 2, 512),      # 12 tiles; 15 memories x 2: a partial row of XCDs
    (2, 6, 2, 128, 320, "bf16", 0, 2, 512),      # three query heads, eight lanes to a slot row
    (9, 16, 16, 128, 320, "bf16", 0, 1, 512),    # 144 memories: one workgroup each, 16 lanes to a slot row
    (9, 16, 16, 128, 576, "bf16", 0, 1, 1024),   # beyond 512 slots
    (11, 9, 9, 128, 1984, "bf16", 0, 2, 1024),   # most loads, 124 tiles for 16 wavefronts
    (5, 32, 16, 128, 448, "bf16", 0, 2, 512),    # two query heads
    (9, 128, 16, 128, 448, "bf16", 0, 1, 512),   # eight, matrix-core read, last block of loads half used
    (2, 35, 5, 64, 704, "bf16", 0, 1, 512),      # seven, 64 columns
    (1, 3, 3, 64, 640, "bf16", 0, 1, 512),
    (2, 4, 4, 128, 64, "f32", 0, 2, 512),
    (9, 32, 16, 128, 256, "f32", 0, 1, 512),     # 32 lanes to a slot row
    (2, 15, 5, 64, 320, "f32", 0, 1, 512),
    (5, 104, 13, 64, 512, "f32", 0, 1, 512),
    (2, 3, 3, 128, 320, "bf16", 1, 1, 512),
    (3, 8, 2, 64, 192, "bf16", 1, 1, 512),
    (2, 6, 2, 128, 192, "f32", 1, 1, 512),
]


@pytest.mark.parametrize("B,Hq,Hkv,d,M,dtype,seq,wgs,threads", CASES)
def test_step_against_oracle_and_streaming(P, R, B, Hq, Hkv, d, M, dtype, seq, wgs, threads):
    """Both, write alone, read alone; step sizes; keys that move, where each sequence has its own."""
    import torch
    w = syn.Workload("whole", 1, B, Hq, Hkv, d, M, dtype, 4)
    ref, gpu, mk, mv, bs = make_pair(w, R.RefCache, P.BctCache, flags=seq, mv0=True)
    _, stream, *_ = make_pair(w, R.RefCache, P.BctCache, flags=seq | P.BCT_STEP_STREAMING, mv0=True)
    assert P.bct_plan_whole(gpu.desc) == (P.BCT_OK, wgs, threads) and P.bct_plan_whole(stream.desc)[1] == 0
    eta = np.abs(syn.unpack(syn.make_step(w, 7)[0], dtype).astype(np.float32))[:, :Hkv, 0].copy()
    dev = lambda a: to_dev(a, dtype)
    gate = torch.from_numpy(eta).to("cuda:0")
    steps = [("both", True, True, None), ("write", False, True, None), ("read", True, False, None), ("gated", True, True, eta)]
    for t, (what, read, write, g) in enumerate(steps):
        q, wq, wv = syn.make_step(w, t)
        q, wq, wv = q if read else None, wq if write else None, wv if write else None
        before = ref.values()
        kw, kg = ({}, {}) if g is None else ({"gate": g}, {"gate": gate})
        o_ref = ref.decode_step(q, wq, wv, **kw)
        outs = []
        for c in (gpu, stream):
            c.set_values(dev(before))
            o = c.decode_step(dev(q), dev(wq), dev(wv), **kg)
            check_state_one_step(to_np(c.values_view(), dtype), ref.values(), dtype, what, before=before)
            outs.append(to_np(o, dtype) if read else None)
        if read:
            for o in outs:
                check_out(o, o_ref, dtype, what)
            # two correct sums of one step: each within two spacings of the oracle's (fp32: 1e-5), so within four
            a, b = (f64(o, dtype) for o in outs)
            worst = np.max(np.abs(a - b), axis=-1)
            peak = np.max(np.abs(b), axis=-1)
            assert np.all(worst <= (2e-5 * peak if dtype == "f32" else 4 * bf16_ulp(peak))), what
    assert np.array_equal(to_np(gpu.keys_view(), dtype), mk)
    if seq:
        q, wq, wv = syn.make_step(w, 9)
        wk = syn.make_step(w, 10)[2]
        kappa = torch.full((B, Hkv), 0.25, device="cuda:0")
        for c in (gpu, stream):
            c.set_values(dev(mv))
            o = c.decode_step_keyed(dev(q), dev(wq), dev(wv), dev(wk), gate=gate, key_gate=kappa)
            check_out(to_np(o, dtype), _keyed(ref, mk, mv, q, wq, wv, wk, eta, 0.25), dtype, "keyed")
            check_state_one_step(to_np(c.values_view(), dtype), ref.values(), dtype, "keyed MV", before=mv)
            check_state_one_step(to_np(c.keys_view(), dtype), ref.keys(), dtype, "keyed MK", before=mk)


def _keyed(ref, mk, mv, q, wq, wv, wk, eta, kappa):
    ref.set_keys(mk)
    ref.set_values(mv)
    return ref.decode_step_keyed(q, wq, wv, wk, gate=eta, kgate=np.full(eta.shape, kappa, np.float32))


# fp32, one query head, 257 to 512 memories of at most 128 slots: one workgroup of 256 threads each (decode_fused_kernel).  Fewest and
# most memories, both widths and both numbers of slots, keys shared and of each sequence
@pytest.mark.parametrize("B,Hkv,d,M,seq", [(257, 1, 64, 64, 0), (32, 16, 64, 128, 0), (20, 15, 128, 64, 1), (64, 8, 128, 128, 0),
                                           (43, 6, 64, 128, 1)])
def test_smallest_caches_own_launch(P, R, B, Hkv, d, M, seq):
    import torch
    w = syn.Workload("fused", 1, B, Hkv, Hkv, d, M, "f32", 4)
    ref, gpu, mk, mv, bs = make_pair(w, R.RefCache, P.BctCache, flags=seq, mv0=True)
    assert P.bct_plan_whole(gpu.desc)[1] == 0 and P.bct_plan_query(gpu.desc)[1]["one_launch"] == 1
    twin = make_pair(w, R.RefCache, P.BctCache, flags=seq, mv0=True)[1]
    eta = syn.make_step(w, 7)[0][:, :, 0].astype(np.float32).copy()   # either sign
    eta[0] = 0.0
    dev = lambda a: to_dev(a, "f32")
    steps = [("both", True, True, None), ("write", False, True, None), ("read", True, False, None), ("gated", True, True, eta)]
    for t, (what, read, write, g) in enumerate(steps):
        q, wq, wv = syn.make_step(w, t)
        q, wq, wv = q if read else None, wq if write else None, wv if write else None
        before = ref.values()
        o_ref = ref.decode_step(q, wq, wv, **({} if g is None else {"gate": g}))
        outs = []
        for c in (gpu, twin):
            c.set_values(dev(before))
            o = c.decode_step(dev(q), dev(wq), dev(wv), **({} if g is None else {"gate": torch.from_numpy(g).cuda()}))
            check_state_one_step(to_np(c.values_view(), "f32"), ref.values(), "f32", what, before=before)
            outs.append(to_np(o, "f32") if read else None)
        if read:
            check_out(outs[0], o_ref, "f32", what)
            assert np.array_equal(outs[0], outs[1])   # repeats itself
        assert np.array_equal(to_np(gpu.values_view(), "f32"), to_np(twin.values_view(), "f32"))
        if not write:
            assert np.array_equal(to_np(gpu.values_view(), "f32"), before)
    assert np.array_equal(to_np(gpu.keys_view(), "f32"), mk)
    if seq:   # a step that writes keys takes the streaming launches
        q, wq, wv = syn.make_step(w, 9)
        wk = syn.make_step(w, 10)[2]
        gpu.set_values(dev(mv))
        o = gpu.decode_step_keyed(dev(q), dev(wq), dev(wv), dev(wk), gate=torch.from_numpy(eta).cuda(),
                                  key_gate=torch.full((B, Hkv), 0.25, device="cuda:0"))
        check_out(to_np(o, "f32"), _keyed(ref, mk, mv, q, wq, wv, wk, eta, 0.25), "f32", "keyed")
        check_state_one_step(to_np(gpu.values_view(), "f32"), ref.values(), "f32", "keyed MV", before=mv)
        check_state_one_step(to_np(gpu.keys_view(), "f32"), ref.keys(), "f32", "keyed MK", before=mk)


def test_repeats_itself_and_graphs(P):
    """Equal inputs give equal bits, launched or replayed."""
    import torch
    for (B, Hq, Hkv, d, M, dtype) in ((3, 16, 4, 128, 320, "bf16"), (4, 40, 40, 128, 256, "bf16"), (2, 4, 4, 64, 64, "f32")):
        w = syn.Workload("whole_bits", 1, B, Hq, Hkv, d, M, dtype, 2)
        cs = []
        for _ in range(2):
            c = P.BctCache(M, B, Hq, Hkv, d, torch.float32 if dtype == "f32" else torch.bfloat16, w.scale, w.scale)
            assert P.bct_plan_whole(c.desc)[1] > 0
            c.set_keys(to_dev(syn.make_keys(w), dtype))
            cs.append(c)
        ins = [to_dev(a, dtype) for a in syn.make_step(w, 0)]
        o = [torch.empty_like(ins[0]) for _ in range(2)]
        graph = torch.cuda.CUDAGraph()
        cs[1].decode_step(*ins, o[1])
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            cs[1].decode_step(*ins, o[1])
        cs[1].set_values(None)
        for _ in range(3):
            cs[0].decode_step(*ins, o[0])
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(o[0].view(torch.uint8), o[1].view(torch.uint8))
            assert torch.equal(cs[0].values_view().view(torch.uint8), cs[1].values_view().view(torch.uint8))


# two workgroups per memory; one already; too long for one (streaming launches); the smallest caches' own launch; re-scored
# with no merge after the pass
@pytest.mark.parametrize("B,Hq,Hkv,d,M,dtype", [(3, 5, 5, 128, 128, "bf16"), (4, 32, 8, 128, 192, "bf16"), (2, 4, 4, 128, 64, "f32"),
                                                (2, 8, 2, 64, 256, "bf16"), (2, 4, 4, 128, 512, "bf16"), (20, 15, 15, 64, 128, "f32"),
                                                (2000, 64, 8, 128, 128, "bf16")])
def test_output_in_the_memory_of_the_inputs(P, R, B, Hq, Hkv, d, M, dtype):
    """out = q, out = the first write query of one head per memory, and rows of others: the results of buffers of their own
    within the criteria of a step."""
    import torch
    w = syn.Workload("whole_alias", 1, B, Hq, Hkv, d, M, dtype, 4)
    few = None if B < 100 else [0, B // 2, B - 1]
    ref, gpu, _, mv, bs = make_pair(w, R.RefCache, P.BctCache, mv0=True, batch_subset=few)
    q, wq, wv = syn.make_step(w, 0)
    dev = lambda a: to_dev(a, dtype)
    sub = lambda a: np.ascontiguousarray(a[bs])
    row = Hq // Hkv * d
    buf = torch.empty(q.size + row, dtype=dev(q).dtype, device="cuda:0")
    cases = [("q", buf[:q.size], buf[:q.size], None), ("shifted", buf[row:], buf[:q.size], None)]
    if Hq == Hkv:
        cases.append(("k_new", None, buf[:q.size], buf[:q.size]))
    for what, qbuf, obuf, kbuf in cases:
        view = lambda b, a: None if b is None else b.view(a.shape).copy_(dev(a))
        before = sub(mv)
        ref.set_values(before)
        gpu.set_values(dev(mv))
        o_ref = ref.decode_step(sub(q), sub(wq), sub(wv))
        dq, dk = view(qbuf, q), view(kbuf, wq)
        o = gpu.decode_step(dev(q) if dq is None else dq, dev(wq) if dk is None else dk, dev(wv), obuf.view(q.shape))
        check_out(to_np(o[bs], dtype), o_ref, dtype, what)
        check_state_one_step(to_np(gpu.values_view()[bs], dtype), ref.values(), dtype, what, before=before)


@pytest.mark.parametrize("B,Hq,Hkv,d,M", [(8, 8, 8, 64, 128), (8, 16, 16, 64, 512), (16, 32, 8, 64, 512), (8, 64, 16, 128, 256)])
def test_fp32_error_is_no_larger_than_the_streaming_launches(P, B, Hq, Hkv, d, M):
    """Root mean square error of the output and the state against 64 bits, over the same 8 steps from the same state."""
    import torch
    w = syn.Workload("whole_error", 1, B, Hq, Hkv, d, M, "f32", 8)
    mk, mv = syn.make_keys(w), syn.make_values0(w)
    k, m0 = mk.astype(np.float64), mv.astype(np.float64)
    soft = lambda s: (lambda e: e / e.sum(-1, keepdims=True))(np.exp(s - s.max(-1, keepdims=True)))
    err = {}
    for name, flags in (("one launch", 0), ("streaming", P.BCT_STEP_STREAMING)):
        c = P.BctCache(M, B, Hq, Hkv, d, torch.float32, w.scale, w.scale, flags)
        assert (P.bct_plan_whole(c.desc)[1] > 0) == (flags == 0)
        c.set_keys(to_dev(mk, "f32"))
        total = np.zeros(2)
        for t in range(8):
            q, wq, wv = syn.make_step(w, t)
            c.set_values(to_dev(mv, "f32"))
            o = to_np(c.decode_step(*(to_dev(a, "f32") for a in (q, wq, wv))), "f32")
            ww = soft(np.einsum("bhd,hmd->bhm", wq.astype(np.float64), k) * w.scale)
            new = m0 + ww[..., None] * wv.astype(np.float64)[:, :, None, :]
            rw = soft(np.einsum("bhgd,hmd->bhgm", q.astype(np.float64).reshape(B, Hkv, -1, d), k) * w.scale)
            out = np.einsum("bhgm,bhmd->bhgd", rw, new).reshape(B, Hq, d)
            total += [np.mean((o - out) ** 2) / np.mean(out ** 2), np.mean((to_np(c.values_view(), "f32") - new) ** 2) / np.mean(new ** 2)]
        err[name] = np.sqrt(total / 8)
    print("rms error out, state", err)
    assert np.all(err["one launch"] <= err["streaming"]), err
