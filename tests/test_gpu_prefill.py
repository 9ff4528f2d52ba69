"""GPU parity of bct_prefill against the oracle's chunk routine (fp32 copy of MV carried
through the chunk, one rounding at its end).

fp32 caches: the chunk is stepped token by token through the decode kernels, so the
decode tolerances apply.  bf16 caches take the MFMA path: softmax weights and the
sub-chunk snapshots of MV enter the read products rounded to bf16 (relative 2^-9 each,
independent over the M slots), which puts the output within a few bf16 ulps of the
output vector's largest entry (asserted at 4) and far inside the 2e-2 absolute bound;
the state uses hi+lo bf16 weights (relative 2^-17) and is held to the one-step decode
criterion: within 1 ulp plus the cancellation allowance, few elements different.
"""
import numpy as np
import pytest

import bct_synth as syn
from _util import bf16_ulp, f64, make_pair, rel_normwise, to_dev, to_np
from test_gpu_parity import check_state_one_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    import paper_2411_15785_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def R():
    from oracle import bct_ref
    return bct_ref


# Relative precision of the write weights on the GPU side of a chunk: hi + lo bf16 split
# (2^-18), fp32 exp2 and normaliser (~2^-21 each), fp32 accumulation inside the MFMA; x2 margin.
PF_WEIGHT_REL = 2.0 ** -16


def prefill_mass(R, ref, mk, wq, T):
    """mass[b][h][m] = sum over the chunk's tokens of ww_t[m], from the oracle itself: the same chunk
    written with wv = 1 into a zero state."""
    dtype = ref.dtype
    aux = R.RefCache(ref.M, ref.B, ref.Hq, ref.Hkv, ref.d, dtype, ref.read_scale, ref.write_scale, ref.flags)
    aux.set_keys(mk)
    ones = syn.pack(np.ones(wq.shape), dtype)
    aux.prefill(None, wq, ones, T)
    return f64(aux.values(), dtype)[..., 0]                         # [B][Hkv][M]


def check_prefill_state(R, ref, mk, wq, wv, got, T, what, mass=None):
    """State after one chunk from a common state.  Each element may differ from the oracle's
    by one rounding flip (1 bf16 ulp) plus the accumulated weight error, which is bounded by
    PF_WEIGHT_REL * sum_t ww_t[m] |wv_t[j]| <= PF_WEIGHT_REL * mass[m] * max_t |wv_t[j]|
    (mass: see prefill_mass; computed here unless the caller already has it)."""
    dtype = ref.dtype
    if mass is None:
        mass = prefill_mass(R, ref, mk, wq, T)
    wvmax = np.max(np.abs(f64(wv, dtype)), axis=1)                  # [B][Hkv][d]
    bound = mass[..., :, None] * wvmax[..., None, :] * 1.01         # mass is itself rounded to bf16
    g, r = f64(got, dtype), f64(ref.values(), dtype)
    d = np.abs(g - r)
    allow = bf16_ulp(r) * 1.0001 + PF_WEIGHT_REL * bound
    assert np.all(d <= allow), f"{what}: bf16 state off by {np.max(d / allow):.2f} x the allowance"
    frac = float(np.mean(got != ref.values()))
    assert frac <= 2e-2, f"{what}: {frac:.2e} of the state elements differ"
    return frac


def check_prefill_out(got, ref, dtype, what, max_ulp=4.0, abs_bound=2e-2):
    """abs_bound=None drops the absolute bound: it is a bound for unit-scale outputs, and where an output
    reaches 4 one bf16 spacing of the output itself is 0.031."""
    g, r = f64(got, dtype), f64(ref, dtype)
    assert np.all(np.isfinite(g)), what
    if dtype == "f32":
        e = rel_normwise(g, r)
        assert e <= 1e-5, f"{what}: fp32 out rel err {e:.3e}"
        return e
    e = float(np.max(np.abs(g - r)))
    assert abs_bound is None or e <= abs_bound, f"{what}: bf16 out abs err {e:.3e}"
    tight = float(np.max(np.max(np.abs(g - r), axis=-1) / bf16_ulp(np.max(np.abs(r), axis=-1))))
    assert tight <= max_ulp, f"{what}: bf16 out {tight:.2f} ulp of the vector max"
    return tight


CASES = [
    # name, B, Hq, Hkv, d, M, dtype, T
    ("f32_small", 2, 4, 2, 64, 128, "f32", 5),
    ("bf16_T128", 2, 2, 2, 128, 256, "bf16", 128),
    ("bf16_ragged200", 2, 4, 2, 128, 256, "bf16", 200),
    ("bf16_T1", 1, 2, 2, 128, 64, "bf16", 1),
    ("bf16_d64_T130", 1, 2, 1, 64, 128, "bf16", 130),
    ("bf16_gqa4_T300", 1, 8, 2, 128, 192, "bf16", 300),
    ("bf16_gqa3_T70", 1, 3, 1, 128, 64, "bf16", 70),
    ("bf16_T512", 1, 2, 2, 128, 1024, "bf16", 512),
    ("bf16_m65536_T64", 1, 1, 1, 128, 65536, "bf16", 64),     # the largest capacity
    ("bf16_m192_T257", 1, 2, 1, 128, 192, "bf16", 257),        # last state workgroup half empty, one token in the last sub-chunk
]


@pytest.mark.parametrize("name,B,Hq,Hkv,d,M,dtype,T", CASES)
@pytest.mark.parametrize("mode", ["rw", "write_only", "read_only"])
def test_prefill_chunk_matches_oracle(P, R, name, B, Hq, Hkv, d, M, dtype, T, mode):
    w = syn.Workload(name, 1, B, Hq, Hkv, d, M, dtype, 0)
    ref, gpu, mk, mv0, _ = make_pair(w, R.RefCache, P.BctCache, mv0=True, max_prefill_T=T)
    for chunk in range(2):   # the second chunk starts from the first one's state
        q, wq, wv = syn.make_step(w, chunk * T, T=T)
        if mode == "write_only":
            q = None
        if mode == "read_only":
            wq = wv = None
        before = ref.values()
        gpu.set_values(to_dev(before, dtype))     # common starting state
        o_ref = ref.prefill(q, wq, wv, T)
        o_gpu = gpu.prefill(to_dev(q, dtype), to_dev(wq, dtype), to_dev(wv, dtype), T)
        what = f"{name}/{mode} chunk {chunk}"
        if mode != "write_only":
            e = check_prefill_out(to_np(o_gpu, dtype), o_ref, dtype, what)
            print(f"{what}: out err {e:.3g}")
        mk_g, mv_g, st = gpu.export()
        assert np.array_equal(to_np(mk_g, dtype), mk)
        if mode == "read_only":
            assert np.array_equal(to_np(mv_g, dtype), before)
        else:
            if dtype == "f32":
                check_state_one_step(to_np(mv_g, dtype), ref.values(), dtype, what)
            else:
                frac = check_prefill_state(R, ref, mk, wq, wv, to_np(mv_g, dtype), T, what)
                print(f"{what}: {frac:.3%} of state elements differ")
        assert st == (chunk + 1) * T == ref.steps


# Edges of the chunk kernels: key tiles of 64 and 128 slots (1 to 5 of them, the last one half), token tiles of 32,
# statistics whose keys are split over one to eight workgroups (row tiles x memories x shares <= 256, 256 slots a
# share), reader wavefronts with no row of the chunk, both head dimensions
@pytest.mark.parametrize("B,Hq,Hkv,d,M,T", [(1, 1, 1, 128, 64, 33), (1, 1, 1, 64, 128, 31), (1, 2, 1, 128, 192, 97),
                                            (2, 2, 2, 128, 320, 160), (1, 1, 1, 128, 512, 129), (1, 4, 4, 64, 832, 65),
                                            (1, 8, 1, 128, 1088, 45), (1, 1, 1, 128, 2112, 20), (3, 5, 5, 64, 2176, 140)])
@pytest.mark.parametrize("mode", ["rw", "write_only", "read_only"])
def test_prefill_tile_edges(P, R, B, Hq, Hkv, d, M, T, mode):
    test_prefill_chunk_matches_oracle(P, R, f"edge_m{M}_t{T}", B, Hq, Hkv, d, M, "bf16", T, mode)


# one to four groups of 32 write tokens asked for in the last sub-chunk (which decides who requests the tiles), one to
# seven tiles, workgroups of one launch with different numbers of them
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,M,T", [(1, 1, 64, 4), (2, 2, 128, 32), (1, 1, 192, 33), (2, 2, 256, 64), (1, 1, 320, 65), (2, 2, 64, 96),
                                        (1, 1, 448, 97), (4, 1, 256, 200), (3, 1, 320, 128), (8, 2, 128, 50)])
def test_prefill_groups_asked_for(P, R, Hq, Hkv, d, M, T):
    test_prefill_chunk_matches_oracle(P, R, "groups", 2, Hq, Hkv, d, M, "bf16", T, "rw")


# Last sub-chunks whose read rows (tokens x query heads of a KV head) fill part of one 128-row tile, exactly one, one and one
# row more, and all G: each launch has as many row tiles as have a row
@pytest.mark.parametrize("Hq,Hkv,d,T", [(8, 1, 128, 4), (8, 1, 64, 15), (16, 2, 128, 16), (8, 1, 64, 17), (16, 2, 64, 130), (8, 1, 128, 144),
                                        (8, 1, 128, 256), (9, 3, 128, 171), (9, 3, 64, 170), (5, 1, 128, 129), (8, 1, 64, 1), (7, 1, 128, 147)])
@pytest.mark.parametrize("mode", ["rw", "read_only"])
def test_prefill_row_tiles_of_the_last_sub_chunk(P, R, Hq, Hkv, d, T, mode):
    test_prefill_chunk_matches_oracle(P, R, f"rows_t{T}", 2, Hq, Hkv, d, 192, "bf16", T, mode)


# Either statistics kernel at the border between them: 384 slots (d = 64: 768) and the next size (one share each), up to 256
# workgroups and more
@pytest.mark.parametrize("B,Hq,Hkv,d,M,T", [(1, 2, 1, 128, 384, 140), (1, 2, 1, 128, 448, 140), (1, 1, 1, 64, 448, 70),
                                            (13, 20, 20, 64, 448, 3), (13, 20, 20, 128, 448, 3), (1, 2, 1, 64, 768, 140),
                                            (1, 2, 1, 64, 832, 140), (13, 20, 20, 64, 832, 3)])
@pytest.mark.parametrize("mode", ["rw", "read_only"])
def test_prefill_statistics_kernels(P, R, B, Hq, Hkv, d, M, T, mode):
    test_prefill_chunk_matches_oracle(P, R, f"stats_m{M}_b{B}", B, Hq, Hkv, d, M, "bf16", T, mode)


# So many KV heads that the write queries of a 32-token tile span 4 GB: the last head count at which a
# 32-bit byte offset reaches them all ((31 * heads * d + d - 8) * 2 < 2^32), and the next one.  Memories are independent, so the oracle
# takes a few of them (62 GB on the device, drawn there).
@pytest.mark.parametrize("Hkv", [541200, 541201])
def test_prefill_write_queries_a_32_bit_offset_apart(P, R, Hkv):
    import torch
    d, M, T = 128, 64, 32
    scale = d ** -0.5
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)

    def draw(*shape):
        return torch.randn(shape, generator=g, dtype=torch.bfloat16, device="cuda:0")

    def some(x, dim):   # of a few heads
        return to_np(torch.stack([x.select(dim, h) for h in (0, 1, 4097, Hkv // 2, Hkv - 2, Hkv - 1)], dim), "bf16")

    gpu = P.BctCache(M, 1, Hkv, Hkv, d, torch.bfloat16, scale, scale, 0, T)
    mk = draw(Hkv, M, d)
    gpu.set_keys(mk)
    mk = some(mk, 0)
    q, wq, wv = (draw(1, T, Hkv, d) for _ in range(3))
    out = some(gpu.prefill(q, wq, wv, T), 2)
    mv = some(gpu.values_view(), 1)
    q, wq, wv = (some(x, 2) for x in (q, wq, wv))
    ref = R.RefCache(M, 1, len(mk), len(mk), d, "bf16", scale, scale, 0)
    ref.set_keys(mk)
    check_prefill_out(out, ref.prefill(q, wq, wv, T), "bf16", f"{Hkv} heads")
    check_prefill_state(R, ref, mk, wq, wv, mv, T, f"{Hkv} heads")


def test_prefill_per_sequence_keys_and_scales(P, R):
    w = syn.Workload("pf_perseq", 1, 2, 4, 2, 128, 128, "bf16", 0)
    T = 96
    ref, gpu, mk, _, _ = make_pair(w, R.RefCache, P.BctCache, flags=1, mv0=True, max_prefill_T=T,
                                   read_scale=0.05, write_scale=0.2)
    q, wq, wv = syn.make_step(w, 0, T=T)
    before = ref.values()
    o_ref = ref.prefill(q, wq, wv, T)
    o_gpu = gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T)
    check_prefill_out(to_np(o_gpu, "bf16"), o_ref, "bf16", "per-seq")
    check_prefill_state(R, ref, mk, wq, wv, to_np(gpu.export()[1], "bf16"), T, "per-seq")


@pytest.mark.parametrize("rs,ws", [(-0.08, 0.09), (0.09, -0.12), (0.0, 0.09), (-0.05, -0.05)])
def test_prefill_and_decode_with_negative_or_zero_scales(P, R, rs, ws):
    """A scale is any finite number: a negative one attends to the least similar keys, zero gives
    uniform weights.  Both entry points against the oracle."""
    w = syn.Workload("pf_neg", 1, 2, 4, 2, 128, 256, "bf16", 0)
    T = 140
    ref, gpu, mk, _, _ = make_pair(w, R.RefCache, P.BctCache, mv0=True, max_prefill_T=T, read_scale=rs, write_scale=ws)
    q, wq, wv = syn.make_step(w, 0, T=T)
    o_ref = ref.prefill(q, wq, wv, T)
    o_gpu = gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T)
    check_prefill_out(to_np(o_gpu, "bf16"), o_ref, "bf16", f"scales {rs} {ws}")
    check_prefill_state(R, ref, mk, wq, wv, to_np(gpu.export()[1], "bf16"), T, f"scales {rs} {ws}")
    before = ref.values()
    gpu.set_values(to_dev(before, "bf16"))
    q, wq, wv = syn.make_step(w, T)
    o_ref = ref.decode_step(q, wq, wv)
    o_gpu = gpu.decode_step(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"))
    assert np.max(np.abs(f64(to_np(o_gpu, "bf16"), "bf16") - f64(o_ref, "bf16"))) <= 2e-2
    check_state_one_step(to_np(gpu.export()[1], "bf16"), ref.values(), "bf16", "decode", before=before)


def test_prefill_then_decode_continues(P, R):
    """A prompt through bct_prefill, then decode steps: the two entry points share one state."""
    w = syn.Workload("pf_dec", 1, 2, 4, 4, 128, 256, "bf16", 0)
    T = 160
    ref, gpu, _, _, _ = make_pair(w, R.RefCache, P.BctCache, max_prefill_T=T)
    q, wq, wv = syn.make_step(w, 0, T=T)
    ref.prefill(q, wq, wv, T)
    gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T)
    for t in range(T, T + 4):
        q, wq, wv = syn.make_step(w, t)
        gpu.set_values(to_dev(ref.values(), "bf16"))
        o_ref = ref.decode_step(q, wq, wv)
        o_gpu = gpu.decode_step(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"))
        assert np.max(np.abs(f64(to_np(o_gpu, "bf16"), "bf16") - f64(o_ref, "bf16"))) <= 2e-2
    assert gpu.steps == T + 4


def test_prefill_argument_errors(P):
    import ctypes
    import torch
    w = syn.Workload("pf_err", 1, 1, 2, 2, 128, 64, "bf16", 0)
    gpu = P.BctCache(w.M, w.B, w.Hq, w.Hkv, w.d, torch.bfloat16, max_prefill_T=8)
    gpu.set_keys(to_dev(syn.make_keys(w), "bf16"))
    L = P.lib()
    q, wq, wv = (to_dev(a, "bf16") for a in syn.make_step(w, 0, T=16))
    out = torch.empty_like(q)
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert L.bct_prefill(gpu._h, p(q), p(wq), p(wv), 16, p(out), s) == P.BCT_ERR_BUFFER_TOO_SMALL  # T > max_prefill_T
    assert L.bct_prefill(gpu._h, p(q), p(wq), p(wv), 0, p(out), s) == P.BCT_ERR_INVALID_ARG
    assert L.bct_prefill(gpu._h, p(q), p(wq), None, 8, p(out), s) == P.BCT_ERR_INVALID_ARG
    assert gpu.steps == 0


@pytest.mark.parametrize("direction", ["rising", "falling"])
def test_prefill_read_rows_whose_maximum_keeps_moving(P, R, direction):
    """Read scores that grow (or fall) steadily along the slot axis, about 12 binary orders per 64-slot tile:
    with "rising" the running maximum of every read row jumps in every tile, so whatever a kernel that
    normalises on the fly has accumulated is rescaled each time; with "falling" the first tile holds the
    maximum and all later weights are tiny.  Keys = ramp * u + small noise, queries = 16.6 * u."""
    w = syn.Workload(f"pf_ramp_{direction}", 1, 2, 2, 2, 64, 512, "bf16", 0)
    T = 70
    ref, gpu, _, _, _ = make_pair(w, R.RefCache, P.BctCache, mv0=True, max_prefill_T=T)
    u = np.ones(w.d) / np.sqrt(w.d)
    ramp = np.arange(w.M) / w.M
    if direction == "falling":
        ramp = ramp[::-1]
    noise = 0.05 * syn.unpack(syn.make_keys(w, 3), "bf16")
    mk = syn.pack(16.0 * ramp[None, :, None] * u[None, None, :] + noise, "bf16")
    ref.set_keys(mk)
    gpu.set_keys(to_dev(mk, "bf16"))
    q, wq, wv = syn.make_step(w, 0, T=T)
    qf = syn.unpack(q, "bf16")
    q = syn.pack(16.6 * u[None, None, None, :] * (1.0 + 0.01 * np.arange(T))[None, :, None, None] + 0.05 * qf, "bf16")
    o_ref = ref.prefill(q, wq, wv, T)
    o_gpu = gpu.prefill(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), T)
    e = check_prefill_out(to_np(o_gpu, "bf16"), o_ref, "bf16", f"ramp {direction}")
    print(f"ramp {direction}: out err {e:.3g}")
