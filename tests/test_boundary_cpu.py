"""CPU-only checks of the C ABI: libbct.so loads without a GPU, exports every symbol
include/bct.h declares, and validates its arguments before the first HIP call."""
import ctypes
import os
import re
import types

import pytest

import paper_2411_15785_amd as P
from paper_2411_15785_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2411_15785_amd import build
        build.build()
    return P.lib()


def declared_functions(header="bct.h", prefix="bct_"):
    src = open(os.path.join(ROOT, "include", header)).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(" + prefix + r"[a-z_]+)\s*\(", src)))


def test_every_declared_symbol_is_exported_and_bound(L):
    names = declared_functions()
    assert {"bct_cache_init", "bct_decode_step", "bct_prefill"} <= set(names)
    aids = declared_functions("bct_measure.h")
    assert {"bct_profile_enable", "bct_profile_read", "bct_stream_copy"} == set(aids) and not set(aids) & set(names)
    names = sorted(names + aids)
    for n in names:
        assert hasattr(L, n), f"{n} is declared in include/ but not exported by libbct.so"
    assert sorted(binding.EXPORTS) == names      # the binding names exactly the header's functions


def test_every_declared_model_symbol_is_exported_and_bound(L):
    from paper_2411_15785_amd import model
    names = declared_functions("bct_model.h", "bctm_")
    assert {"bctm_linear", "bctm_swiglu", "bctm_rmsnorm", "bctm_embed", "bctm_argmax", "bctm_pack_weight", "bctm_pack_rows"} <= set(names)
    ML = model.mlib()
    for n in names:
        assert hasattr(ML, n), f"{n} is declared in include/bct_model.h but not exported by libbct.so"
    assert sorted(model.MODEL_EXPORTS) == names


def test_model_entry_points_check_arguments_before_touching_the_gpu(L):
    from paper_2411_15785_amd import model
    ML = model.mlib()
    p = ctypes.c_void_p
    a, b, c = p(0x10000), p(0x20000), p(0x30000)
    assert ML.bctm_linear(a, b, None, c, 4, 72, 32, 0, None) == P.BCT_ERR_UNSUPPORTED       # K % 32
    assert ML.bctm_linear(a, b, None, c, 4, 64, 40, 0, None) == P.BCT_ERR_UNSUPPORTED       # N % 16
    assert ML.bctm_pack_weight(a, b, 40, 64, None) == P.BCT_ERR_UNSUPPORTED
    assert ML.bctm_pack_weight(a, a, 32, 64, None) == P.BCT_ERR_INVALID_ARG              # in place
    assert ML.bctm_pack_weight(a, None, 32, 64, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_linear(a, None, None, c, 4, 64, 32, 0, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_linear(a, b, None, c, 0, 64, 32, 0, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_linear(p(0x10008), b, None, c, 4, 64, 32, 0, None) == P.BCT_ERR_MISALIGNED
    assert ML.bctm_linear(a, b, p(0x40004), c, 4, 64, 32, 0, None) == P.BCT_ERR_MISALIGNED
    assert ML.bctm_swiglu(a, b, None, c, 4, 64, 32, 0, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_rmsnorm(a, b, c, 4, 12, 1e-5, 0, None) == P.BCT_ERR_UNSUPPORTED          # dim % 8
    assert ML.bctm_rmsnorm(a, b, c, 4, 32768, 1e-5, 0, None) == P.BCT_ERR_UNSUPPORTED
    assert ML.bctm_rmsnorm(a, b, c, 4, 40, 1e-5, 2, None) == P.BCT_ERR_UNSUPPORTED           # tiled: dim % 32
    assert ML.bctm_rmsnorm(a, b, a, 4, 64, 1e-5, 2, None) == P.BCT_ERR_INVALID_ARG           # tiled in place
    assert ML.bctm_rmsnorm(a, b, c, 4, 64, 1e-5, 1, None) == P.BCT_ERR_INVALID_ARG           # not its flag
    assert ML.bctm_linear(a, b, None, c, 4, 64, 32, 2, None) == P.BCT_ERR_INVALID_ARG        # no tiled output
    assert ML.bctm_linear(a, b, None, a, 4, 64, 32, 0, None) == P.BCT_ERR_INVALID_ARG        # out is x
    assert ML.bctm_swiglu(a, b, b, c, 4, 64, 48, 2, None) == P.BCT_ERR_UNSUPPORTED           # tiled out: N % 32
    assert ML.bctm_swiglu(a, b, b, c, 4, 64, 32, 8, None) == P.BCT_ERR_INVALID_ARG
    d = p(0x50000)
    assert ML.bctm_linear_split(a, b, c, 32, d, 24, None, 0, 4, 64, 0, None) == P.BCT_ERR_UNSUPPORTED   # width % 16
    assert ML.bctm_linear_split(a, b, c, 32, None, 16, None, 0, 4, 64, 0, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_linear_split(a, b, c, 32, d, 16, None, 16, 4, 64, 0, None) == P.BCT_ERR_INVALID_ARG  # out2 missing
    assert ML.bctm_linear_split(a, b, c, 0, d, 16, None, 0, 4, 64, 0, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_pack_rows(a, b, 4, 40, None) == P.BCT_ERR_UNSUPPORTED
    assert ML.bctm_pack_rows(a, a, 4, 64, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_embed(None, b, c, 4, 10, 64, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_embed(a, b, c, 4, 10, 12, None) == P.BCT_ERR_UNSUPPORTED
    assert ML.bctm_argmax(a, None, 4, 10, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_last_error().decode() != ""


def test_projection_kernel_choice():
    """bctm_linear_plan: which kernel a projection shape runs in (host logic).  The 7B-shaped stack: a decode
    batch streams the weights; a prompt chunk takes the matrix-core kernel (its tile: test_projection_tile)."""
    from paper_2411_15785_amd import model as Mo
    S, SW, T128, T256 = (Mo.BCTM_KERNEL_STREAMING, Mo.BCTM_KERNEL_STREAMING_WIDE, Mo.BCTM_KERNEL_TILE128,
                         Mo.BCTM_KERNEL_TILE256)
    plan = Mo.bctm_linear_plan
    # decode batch of 32
    assert plan(32, 4096, 12288) == Mo.BCTM_KERNEL_STREAMING_TRIPLE and plan(32, 4096, 4096) == S
    assert plan(32, 11008, 4096) == S and plan(32, 4096, 6144) == S and plan(32, 4096, 12304) == S
    assert plan(32, 4096, 32000) == SW and plan(32, 4096, 11008, swiglu=True) == S
    assert plan(127, 4096, 4096) == S
    # prompt chunk of 32 x 512 rows
    for N in (12288, 4096, 32000):
        assert plan(16384, 4096, N) == T256
    assert plan(16384, 4096, 11008, swiglu=True) == T256
    # in between, and feature counts the larger tiles do not divide
    assert plan(128, 4096, 4096) == T128 and plan(1023, 4096, 4096) == T128 and plan(1024, 4096, 4096) == T256
    assert plan(4096, 4096, 384) == T128 and plan(4096, 4096, 192, swiglu=True) == T128
    assert plan(4096, 4096, 48) == S and plan(4096, 4096, 96, swiglu=True) == S
    assert plan(4096, 4096, 16416) == SW
    ML = Mo.mlib()
    k = ctypes.c_uint32(0)
    assert ML.bctm_linear_plan(4, 72, 32, 0, ctypes.byref(k)) == P.BCT_ERR_UNSUPPORTED
    assert ML.bctm_linear_plan(4, 64, 32, 0, None) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_linear_plan(0, 64, 32, 0, ctypes.byref(k)) == P.BCT_ERR_INVALID_ARG


def test_projection_tile():
    """bctm_linear_tile: rows x features per workgroup and the parts that K is summed in, as launched (host logic)."""
    from paper_2411_15785_amd import model as Mo
    tile = Mo.bctm_linear_tile
    # streaming: row tiles of 16; 1, 2 or 3 feature tiles; K over the workgroup's wavefronts
    assert tile(4, 11008, 4096) == (16, 16, 16) and tile(17, 11008, 4096) == (32, 16, 16)
    assert tile(16, 4096, 32000) == (16, 32, 8) and tile(127, 4096, 32000) == (32, 32, 8)
    assert tile(8, 4096, 12288) == (16, 48, 8) and tile(9, 4096, 12288) == (32, 48, 8)
    assert tile(9, 4096, 12288, tiled=True) == (16, 48, 8) and tile(9, 4096, 14400) == (16, 48, 8)
    assert tile(16, 4096, 11008, swiglu=True) == (16, 16, 4) and tile(32, 4096, 11008, swiglu=True) == (32, 16, 4)
    assert tile(4096, 4096, 96, swiglu=True) == (32, 16, 4)
    # the matrix-core kernel's tiles (128 x 512: below), plain and SwiGLU (half as many features of two matrices)
    assert tile(128, 4096, 128) == (64, 64, 2) and tile(640, 11008, 4096) == (128, 128, 2)
    assert tile(1024, 4096, 4096) == (128, 128, 2) and tile(1030, 4096, 4096) == (128, 256, 1)
    assert tile(640, 4096, 12288) == (128, 256, 1) and tile(1000, 4096, 32768) == (256, 256, 1)
    assert tile(1030, 4096, 4224) == (128, 128, 1) and tile(16384, 11008, 4096) == (256, 256, 1)
    assert tile(16384, 4096, 11008, swiglu=True) == (256, 128, 1) and tile(128, 4096, 64, swiglu=True) == (64, 32, 2)
    ML = Mo.mlib()
    k = [ctypes.byref(ctypes.c_uint32(0)) for _ in range(3)]
    assert ML.bctm_linear_tile(4, 72, 32, 0, 0, *k) == P.BCT_ERR_UNSUPPORTED
    assert ML.bctm_linear_tile(0, 64, 32, 0, 0, *k) == P.BCT_ERR_INVALID_ARG
    assert ML.bctm_linear_tile(4, 64, 32, 0, 0, k[0], None, k[2]) == P.BCT_ERR_INVALID_ARG


def test_projection_tile_of_512_features():
    """128 x 512 against 256 x 256: for tiled inputs of more than 4096 only where it saves a round of five or fewer; K is summed in as
    many parts for either order of x."""
    from paper_2411_15785_amd import model as Mo
    tile = Mo.bctm_linear_tile
    for rows, K, N, swiglu in [(1658, 8192, 24576, True), (1642, 8192, 47616, False), (4654, 11008, 20992, False),
                               (2149, 5120, 37888, False), (5969, 11008, 6912, True), (4654, 4128, 20992, False)]:
        per = 2 if swiglu else 1
        assert tile(rows, K, N, swiglu, tiled=True) == (256, 256 // per, 1)
        assert tile(rows, K, N, swiglu) == (128, 512 // per, 1)
        assert tile(rows, 4096, N, swiglu, tiled=True) == (128, 512 // per, 1)
    for rows, K, N, swiglu in [(2135, 11008, 14592, True), (4948, 8192, 13312, False), (838, 11008, 53248, False), (319, 8192, 69632, False)]:
        assert tile(rows, K, N, swiglu, tiled=True) == tile(rows, K, N, swiglu) == (128, 256 if swiglu else 512, 1)
    for rows in range(128, 9000, 61):
        for N in range(256, 40000, 1280):
            for K in (4096, 8192):
                for swiglu in (False, True):
                    assert tile(rows, K, N, swiglu, tiled=True)[2] == tile(rows, K, N, swiglu)[2]


def desc(**kw):
    d = dict(capacity_M=4096, batch=32, n_q_heads=32, n_kv_heads=32, head_dim=128, dtype=P.BCT_BF16,
             read_scale=0.0884, write_scale=0.0884, flags=0)
    d.update(kw)
    return P.make_desc(**d)


def test_query_sizes_are_exact_and_constant(L):
    st, cb, wb = P.bct_cache_query(desc(), 0)
    assert st == P.BCT_OK
    assert cb == 32 * 4096 * 128 * 2 + 32 * 32 * 4096 * 128 * 2      # MK + MV, nothing else
    st, cb2, wb2 = P.bct_cache_query(desc(), 512)
    assert st == P.BCT_OK and cb2 == cb and wb2 > wb                # prefill only adds workspace
    st, cbp, _ = P.bct_cache_query(desc(flags=P.BCT_MK_PER_SEQUENCE), 0)
    assert st == P.BCT_OK and cbp == 2 * 32 * 32 * 4096 * 128 * 2
    st, cbf, _ = P.bct_cache_query(desc(dtype=P.BCT_F32, head_dim=64, capacity_M=64, batch=1, n_q_heads=4,
                                        n_kv_heads=4), 0)
    assert st == P.BCT_OK and cbf == 2 * 4 * 64 * 64 * 4


@pytest.mark.parametrize("kw,status", [
    (dict(capacity_M=0), P.BCT_ERR_INVALID_ARG),
    (dict(batch=0), P.BCT_ERR_INVALID_ARG),
    (dict(n_q_heads=30), P.BCT_ERR_INVALID_ARG),            # not a multiple of n_kv_heads
    (dict(read_scale=float("nan")), P.BCT_ERR_INVALID_ARG),
    (dict(capacity_M=100), P.BCT_ERR_UNSUPPORTED),          # not a multiple of 64
    (dict(capacity_M=131072), P.BCT_ERR_UNSUPPORTED),
    (dict(head_dim=96), P.BCT_ERR_UNSUPPORTED),
    (dict(dtype=7), P.BCT_ERR_UNSUPPORTED),
    (dict(flags=8), P.BCT_ERR_UNSUPPORTED),
    (dict(flags=4), P.BCT_ERR_UNSUPPORTED),
    (dict(n_q_heads=32, n_kv_heads=2), P.BCT_ERR_UNSUPPORTED),   # 16 query heads per KV head
])
def test_bad_descriptors_are_rejected(L, kw, status):
    st, _, _ = P.bct_cache_query(desc(**kw), 0)
    assert st == status
    assert P.bct_last_error() != ""
    st, h = P.bct_cache_init(desc(**kw), 0, ctypes.c_void_p(0x1000), 1 << 40, ctypes.c_void_p(0x2000), 1 << 40, None)
    assert st == status and not h.value


def test_init_checks_pointers_and_sizes_before_touching_the_gpu(L):
    d = desc()
    _, cb, wb = P.bct_cache_query(d, 0)
    ok_c, ok_w = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x20000)
    assert L.bct_cache_query(None, 0, None, None) == P.BCT_ERR_INVALID_ARG
    assert P.bct_cache_init(d, 0, None, cb, ok_w, wb, None)[0] == P.BCT_ERR_INVALID_ARG
    assert P.bct_cache_init(d, 0, ok_c, cb, None, wb, None)[0] == P.BCT_ERR_INVALID_ARG
    assert P.bct_cache_init(d, 0, ctypes.c_void_p(0x10010), cb, ok_w, wb, None)[0] == P.BCT_ERR_MISALIGNED
    assert P.bct_cache_init(d, 0, ok_c, cb - 1, ok_w, wb, None)[0] == P.BCT_ERR_BUFFER_TOO_SMALL
    assert P.bct_cache_init(d, 0, ok_c, cb, ok_w, wb - 1, None)[0] == P.BCT_ERR_BUFFER_TOO_SMALL
    assert P.bct_cache_init(d, 512, ok_c, cb, ok_w, wb, None)[0] == P.BCT_ERR_BUFFER_TOO_SMALL  # prefill needs more


def test_null_handles_and_messages(L):
    vp = ctypes.c_void_p
    assert L.bct_decode_step(None, vp(16), vp(16), vp(16), vp(16), None) == P.BCT_ERR_INVALID_ARG
    assert L.bct_prefill(None, vp(16), vp(16), vp(16), 4, vp(16), None) == P.BCT_ERR_INVALID_ARG
    assert L.bct_cache_set_keys(None, vp(16), None) == P.BCT_ERR_INVALID_ARG
    assert L.bct_cache_steps(None, None) == P.BCT_ERR_INVALID_ARG
    assert L.bct_stream_copy(vp(16), vp(16), 24, None) == P.BCT_ERR_INVALID_ARG   # not a multiple of 16
    assert L.bct_stream_copy(vp(8), vp(16), 32, None) == P.BCT_ERR_MISALIGNED
    L.bct_cache_destroy(None)                                                     # harmless
    for st in range(7):
        assert P.bct_strerror(st) not in ("", "unknown status")
    assert P.bct_strerror(99) == "unknown status"


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "one GPU" in r.stderr


def test_launch_plans_of_the_five_workloads(L):
    """Host logic: which path a decode step takes, decided from the descriptor alone."""
    import bct_synth as syn

    def plan(name, flags=0):
        w = syn.WORKLOADS[name]
        dt = P.BCT_F32 if w.dtype == "f32" else P.BCT_BF16
        st, info = P.bct_plan_query(P.make_desc(w.M, w.B, w.Hq, w.Hkv, w.d, dt, w.scale, w.scale, flags))
        assert st == P.BCT_OK
        return info

    c1 = plan("cfg1")            # 4 memories of 64 slots: one launch
    assert c1["one_launch"] == 1 and c1["launches"] == 1
    c1s = plan("cfg1", P.BCT_STEP_STREAMING)
    assert c1s["one_launch"] == 0 and c1s["scores_mfma"] == 0 and c1s["launches"] == 2     # one split: no merge
    c2 = plan("cfg2")            # M = 1024: too large for the one-launch step; 256 memories of 256 KB: one MV-pass workgroup each
    assert c2["one_launch"] == 0 and c2["scores_mfma"] == 1
    assert c2["mv_workgroup"] == 1024 and c2["mv_loads_per_lane"] == 16 and c2["mv_splits"] == 1 and c2["launches"] == 2
    w2 = syn.WORKLOADS["cfg2"]
    for batch, splits in ((4, 16), (5, 16), (6, 1), (8, 1), (9, 16)):     # 128, 160: too few memories; 288 x 256 KB: too much in all
        st, pl = P.bct_plan_query(P.make_desc(w2.M, batch, w2.Hq, w2.Hkv, w2.d, P.BCT_BF16, w2.scale, w2.scale))
        assert st == P.BCT_OK and pl["mv_splits"] == splits, (batch, pl)
    c3 = plan("cfg3")            # the headline shape: scores, MV pass (merging the 32 partials per row itself), merge
    assert c3 == dict(launches=3, one_launch=0, scores_mfma=1, slots_per_stat=128, normaliser_launch=0,
                      mv_workgroup=256, mv_loads_per_lane=4, mv_splits=64)
    assert c3["mv_workgroup"] * c3["mv_loads_per_lane"] * 16 * c3["mv_splits"] == 4096 * 128 * 2   # one memory, one-shot
    c4 = plan("cfg4")            # 4 query heads per KV head: the MFMA read, 16 KB workgroups; 128 partials per row: own launch
    assert c4["mv_workgroup"] == 128 and c4["mv_loads_per_lane"] == 8 and c4["normaliser_launch"] == 1
    w4 = syn.WORKLOADS["cfg4"]
    st, f4 = P.bct_plan_query(P.make_desc(w4.M, w4.B, w4.Hq, w4.Hkv, w4.d, P.BCT_F32, w4.scale, w4.scale))
    assert st == P.BCT_OK and f4["mv_workgroup"] == 512          # fp32 storage keeps the vector-ALU read
    assert c4["launches"] == 4
    # scores again in the MV pass: several query heads, bf16, d = 128, shared keys, 192 MB of scores and partial outputs
    # (per workgroup of 64 slots 256 (1 + G) + 512 G bytes), 2.5 MB of keys on an XCD (1 / gcd(splits x heads, 8) of them)
    def again(M, B, G, d=128, dt=P.BCT_BF16, flags=0, H=8):
        st, v = P.bct_plan_rescores(P.make_desc(M, B, H * G, H, d, dt, 0.1, 0.1, flags))
        assert st == P.BCT_OK
        return v
    assert again(8192, 64, 4) == 1 and again(8192, 60, 4) == 1 and again(8192, 59, 4) == 0 and again(8192, 16, 4) == 0
    assert again(64, 10922, 8) == 0 and again(64, 10923, 8) == 1                 # no partial outputs: one split
    assert again(10240, 64, 8) == 1 and again(10304, 64, 8) == 0                 # 2.5 MB of keys on an XCD
    assert again(8192, 64, 8, H=7) == 1 and again(8128, 64, 8, H=7) == 0         # 1/8 of the keys; all of them
    assert again(4992, 101, 8, H=7) == 0 and again(4992, 101, 8, H=4) == 1        # half of 9 MB; 1/8 of 5 MB
    assert again(8192, 64, 2) == 0 and again(8192, 64, 4, d=64) == 0 and again(8192, 64, 4, dt=P.BCT_F32) == 0
    assert again(8192, 64, 4, flags=P.BCT_MK_PER_SEQUENCE) == 0
    assert P.bct_plan_rescores(desc(capacity_M=100))[0] == P.BCT_ERR_UNSUPPORTED
    assert L.bct_plan_rescores(ctypes.byref(desc()), None) == P.BCT_ERR_INVALID_ARG
    c5 = plan("cfg5")            # 128 partials per row, two per lane of the MV pass: no normaliser launch
    assert c5["slots_per_stat"] == 128 and c5["normaliser_launch"] == 0 and c5["launches"] == 3
    c5 = plan("cfg5")
    assert c5["mv_splits"] * c5["mv_workgroup"] * c5["mv_loads_per_lane"] * 16 == 16384 * 128 * 2
    assert plan("cfg3", P.BCT_MK_PER_SEQUENCE)["scores_mfma"] == 0      # per-sequence keys: no shared contraction
    st, _ = P.bct_plan_query(desc(capacity_M=100))
    assert st == P.BCT_ERR_UNSUPPORTED
    assert L.bct_plan_query(ctypes.byref(desc()), None) == P.BCT_ERR_INVALID_ARG


class _TorchOfTwoDevices:
    """As much of torch as a launch asks for: two devices, stream 100 + i current on device i."""

    def __init__(self, private):
        self.current, self.entered = 0, []
        outer = self

        class Device:
            def __init__(self, device):
                self.to = outer.current if device.index is None else device.index

            def __enter__(self):
                outer.entered.append(self.to)
                self.back, outer.current = outer.current, self.to

            def __exit__(self, *_):
                outer.current = self.back

        def stream(index):
            return 100 + index
        self._C = types.SimpleNamespace(**({"_cuda_getCurrentRawStream": stream} if private else {}))
        self.cuda = types.SimpleNamespace(device=Device, current_device=lambda: outer.current,
                                          current_stream=lambda index: types.SimpleNamespace(cuda_stream=stream(index)))


@pytest.mark.parametrize("private", [True, False])
def test_launches_go_to_the_device_of_their_tensors(monkeypatch, private):
    """_launch, without a GPU: the device that is current is not entered, another one is, and left again however the call
    ends; the stream is the called device's; a torch without the private function serves as well."""
    torch = _TorchOfTwoDevices(private)
    monkeypatch.setattr(binding, "_torch_module", torch)
    monkeypatch.setattr(binding, "_raw_stream", binding._raw_stream_of(torch))
    dev = lambda index: types.SimpleNamespace(type="cuda", index=index)
    seen = lambda *args: (torch.current, args)
    assert binding._launch(seen, dev(0), 7, None) == (0, (7, None, 100)) and torch.entered == []
    assert binding._launch(seen, dev(1), 7) == (1, (7, 101)) and torch.entered == [1] and torch.current == 0
    assert binding._launch(seen, dev(None)) == (0, (100,)) and torch.entered == [1, 0]
    with pytest.raises(ZeroDivisionError):
        binding._launch(lambda s: 1 // 0, dev(1))
    assert torch.current == 0
    torch.current = 1
    assert binding._stream_ptr() == 101
    assert binding._launch(seen, dev(0)) == (0, (100,)) and torch.current == 1


def test_every_pointer_parameter_is_declared(L):
    """Pointers go to the library as plain integers, which ctypes cuts to 32 bits where no argument type is declared."""
    from paper_2411_15785_amd import model
    ML = model.mlib()
    assert [n for n in binding.EXPORTS + model.MODEL_EXPORTS if getattr(ML, n).argtypes is None] == []


def test_projection_of_ragged_feature_counts():
    """Feature counts that no tile divides: the matrix-core kernel beyond a round of streaming workgroups (two of long sums)."""
    from paper_2411_15785_amd import model as Mo
    S, T128, plan = Mo.BCTM_KERNEL_STREAMING, Mo.BCTM_KERNEL_TILE128, Mo.bctm_linear_plan
    assert plan(709, 11264, 2912) == T128 and plan(1500, 4000, 1504, swiglu=True) == T128 and plan(127, 4096, 12336) == S + 4
    assert plan(256, 3072, 512 + 16) == T128 and plan(256, 3072, 496) == S          # 264 and 248 workgroups
    assert plan(256, 3104, 1024 + 16) == T128 and plan(256, 3104, 1008) == S        # 520 and 504: streaming is the faster up to there
    assert plan(145, 4032, 1200) == S and plan(360, 7072, 448) == S
    assert plan(256, 11008, 1024 + 16) == T128 and plan(256, 11008, 1008) == S      # 520 and 504
    assert plan(256, 11008, 544, swiglu=True) == T128 and plan(256, 11008, 480, swiglu=True) == S
    assert plan(4096, 4096, 112) == S and plan(4096, 4096, 144) == T128             # at least one tile of features
    assert plan(4096, 4096, 16384) == Mo.BCTM_KERNEL_TILE256 and plan(4096, 4096, 16400) == S
    tile = Mo.bctm_linear_tile   # so the parts that K is summed in follow from rows, N and K
    assert tile(256, 3072, 736)[2] == 2 and tile(256, 3104, 736)[2] == 16 and tile(256, 3104, 736, swiglu=True)[2] == 2


def test_workgroups_of_the_mv_pass_cover_every_memory(L):
    """Plans of streaming steps: splits of a memory x slots of a workgroup are M slots and no workgroup more; where the scores
    are made again a workgroup has one tile of slots or two, and only keys that the batch shares are scored again.  Several heads
    with 64 columns: up to four."""
    import itertools
    rescored = 0
    heads = [(8192, 64, 8), (8192, 32, 8), (4096, 64, 16), (2048, 64, 16), (1280, 1020, 3), (1344, 1000, 3), (128, 2000, 8),
             (192, 2001, 8), (64, 10923, 8), (15360, 24, 1), (16384, 64, 16), (640, 3, 2)]
    for (M, B, H), G, d, dt, keys in itertools.product(heads, range(1, 9), (64, 128), (P.BCT_F32, P.BCT_BF16),
                                                       (0, P.BCT_MK_PER_SEQUENCE)):
        dsc = P.make_desc(M, B, H * G, H, d, dt, 0.1, 0.1, keys | P.BCT_STEP_STREAMING)
        (st, plan), (st2, again) = P.bct_plan_query(dsc), P.bct_plan_rescores(dsc)
        assert st == st2 == P.BCT_OK
        row = d * (4 if dt == P.BCT_F32 else 2)
        tile = plan["mv_workgroup"] * plan["mv_loads_per_lane"] * 16 // row
        tiles = -(-M // tile)
        what = (M, B, H, G, d, dt, keys, plan, again)
        per = (1, 2) if again else (1, 2, 3, 4) if d == 64 and dt == P.BCT_BF16 and G > 2 else (1,)
        assert plan["mv_splits"] in [-(-tiles // n) for n in per], what
        assert not again or not keys, what
        rescored += again
    assert rescored > 0


def test_route_of_a_step_whose_output_overlaps_its_inputs(L):
    """A one-launch step stores its output rows while other workgroups may still read theirs: where `out` shares memory with
    an input it is taken only for the same rows, by one workgroup per memory."""
    def route(M, B, G, d, dt, flags=0, H=4, **at):
        st, wgs, splits = P.bct_plan_step(P.make_desc(M, B, H * G, H, d, dt, 0.1, 0.1, flags), **at)
        assert st == P.BCT_OK
        return wgs, splits
    a, far = 1 << 32, dict(k_new=1 << 33, v_new=3 << 32)
    for dt, d, G, two in ((P.BCT_BF16, 128, 1, 2), (P.BCT_BF16, 128, 4, 2), (P.BCT_F32, 128, 1, 2), (P.BCT_BF16, 64, 4, 1),
                          (P.BCT_F32, 64, 1, 1)):
        row = d * (4 if dt == P.BCT_F32 else 2)
        out_bytes, kv_bytes = 2 * 4 * G * row, 2 * 4 * row
        go = lambda **at: route(128, 2, G, d, dt, out=a, **at)[0]
        assert go(q=2 * a, **far) == two and go(q=None, **far) == two
        assert go(q=a, **far) == 1                                            # out is q
        assert go(q=a + 16, **far) == 0 and go(q=a - 16, **far) == 0          # other rows of it
        assert go(q=a + out_bytes, **far) == two and go(q=a - out_bytes, **far) == two
        for name in ("k_new", "v_new"):
            at = dict(far, q=2 * a)
            assert go(**dict(at, **{name: a})) == (1 if G == 1 else 0)
            assert go(**dict(at, **{name: a + out_bytes - 16})) == 0 and go(**dict(at, **{name: a + 16 - kv_bytes})) == 0
            assert go(**dict(at, **{name: a + out_bytes})) == two and go(**dict(at, **{name: a - kv_bytes})) == two
        assert go(q=2 * a, gate=a + out_bytes - 4, **far) == 0 and go(q=2 * a, gate=a + out_bytes, **far) == two
    own = P.BCT_MK_PER_SEQUENCE
    keyed = dict(far, q=a, out=a, key_new=5 << 32)
    assert route(256, 2, 1, 64, P.BCT_BF16, own, **keyed)[0] == 1
    assert route(256, 2, 1, 64, P.BCT_BF16, own, **dict(keyed, key_new=a + 16))[0] == 0
    assert route(256, 2, 1, 64, P.BCT_BF16, own, **dict(keyed, key_gate=a))[0] == 0
    # the smallest caches' own launch: 300 memories, fp32, one query head
    assert route(64, 75, 1, 64, P.BCT_F32, q=a, out=a, **far)[0] == 1 and route(64, 75, 1, 64, P.BCT_F32, q=a + 16, out=a, **far)[0] == 0
    # one workgroup per memory would be a longer chain than the streaming launches: those
    assert route(512, 2, 1, 128, P.BCT_BF16, q=2 * a, out=a, **far)[0] == 2 and route(512, 2, 1, 128, P.BCT_BF16, q=a, out=a, **far)[0] == 0
    # no merge after the pass: it reads q and k_new itself where it scores again, so two splits for rows of others
    big = dict(out=a, **far)
    assert route(128, 2000, 8, 128, P.BCT_BF16, H=8, q=a, **big) == (0, 1) and route(128, 2000, 8, 128, P.BCT_BF16, H=8, q=a + 16, **big) == (0, 2)
    dsc = P.make_desc(128, 2000, 64, 8, 128, P.BCT_BF16, 0.1, 0.1, 0)
    one = P.make_desc(128, 2000, 64, 8, 128, P.BCT_BF16, 0.1, 0.1, P.BCT_MK_PER_SEQUENCE)   # two splits always
    assert P.bct_cache_query(dsc, 0)[2] == P.bct_cache_query(one, 0)[2]   # the scratch for two is there
    assert P.bct_plan_step(None, 0)[0] == P.BCT_ERR_INVALID_ARG


def test_scratch_of_several_heads_with_64_columns(L):
    """Tiles of 128 slots a workgroup: one, two or three by the number of tiles, more where a step's scratch then passes the static
    array and up to four stay inside it: the first that fits.  Every cache that fits with 512 slots does."""
    import itertools
    up = lambda n: -(-n // 256) * 256
    wider = 0
    for G, units, M in itertools.product(range(3, 9), (1, 2, 5, 7, 16, 24, 31, 64, 100, 435), [64 * m for m in range(1, 1025)]):
        rows = units * (1 + G)
        rest = up(rows * M * 4) + up(rows * (M // 32) * 8) + up(rows * 8)
        need = lambda per: rest + up(-(-(-(-M // 128)) // per) * units * G * 64 * 4)
        limit = 8 << 20
        if need(1) > limit + (1 << 21):
            break
        dsc = P.make_desc(M, 1, units * G, units, 64, P.BCT_BF16, 0.1, 0.1, P.BCT_STEP_STREAMING)
        w = units * -(-M // 128)
        few = 2 if 2560 < w <= 3456 else 3 if 3456 < w <= 4096 else 1
        per = next((n for n in range(few, 5) if need(n) <= limit), few)
        assert need(per) <= limit or need(4) > limit
        wider += per > few
        assert P.bct_cache_query(dsc, 0)[2] == need(per), (G, units, M)
        assert P.bct_plan_query(dsc)[1]["mv_splits"] == -(-(-(-M // 128)) // per), (G, units, M)
    assert wider > 50


def test_odd_memories_of_64_columns_read_on_the_vector_alu(L):
    """Three or four heads, bf16, 64 columns, M an odd multiple of 64, long memories and much of them: workgroups of 512 slots."""
    def threads(M, n, G, d=64, dt=P.BCT_BF16, keys=0):
        st, plan = P.bct_plan_query(P.make_desc(M, 1, n * G, n, d, dt, 0.1, 0.1, keys))
        assert st == P.BCT_OK and plan["mv_splits"] * plan["mv_workgroup"] * plan["mv_loads_per_lane"] * 16 >= M * d * (2 if dt == P.BCT_BF16 else 4)
        return plan["mv_workgroup"]
    for keys in (0, P.BCT_MK_PER_SEQUENCE):
        assert threads(10304, 820, 3, keys=keys) == 512 and threads(10240, 820, 3, keys=keys) == 128
    assert threads(7104, 880, 3) == 512 and threads(7104, 879, 3) == 128 and threads(6976, 2000, 3) == 128
    assert threads(14144, 663, 4) == 512 and threads(14144, 662, 4) == 128 and threads(13888, 900, 4) == 128
    assert threads(14144, 900, 5) == 128 and threads(14144, 900, 3, d=128) == 128


def test_where_the_one_launch_steps_begin_and_end(L):
    """fp32, one query head, 257 to 512 memories of at most 128 slots: the smallest caches' own launch; below and beside it the
    whole-step launch (workgroups per memory, threads), beyond both the streaming launches."""
    def form(M, n, G, d, dt, keys=0):
        dsc = P.make_desc(M, 1, n * G, n, d, dt, 0.1, 0.1, keys)
        (st, wgs, threads), (st2, plan) = P.bct_plan_whole(dsc), P.bct_plan_query(dsc)
        assert st == st2 == P.BCT_OK and (plan["launches"] == 1) == (plan["one_launch"] == 1)
        if wgs:
            assert plan["one_launch"] == 1 and threads in (512, 1024)
            return wgs, threads
        return "own" if plan["one_launch"] else "streaming"
    F, B = P.BCT_F32, P.BCT_BF16
    for d in (64, 128):
        for M in (64, 128):
            for keys in (0, P.BCT_MK_PER_SEQUENCE):
                assert form(M, 256, 1, d, F, keys) == (1, 512) and form(M, 257, 1, d, F, keys) == "own"
                assert form(M, 512, 1, d, F, keys) == "own" and form(M, 513, 1, d, F, keys) == "streaming"
                assert form(M, 512, 2, d, F, keys) == (1, 512) and form(M, 513, 2, d, F, keys) == "streaming"
                assert form(M, 1024, 4, d, F, keys) == (1, 512) and form(M, 1025, 4, d, F, keys) == "streaming"
                assert form(M, 640, 1, d, B, keys) == (1, 512) and form(M, 641, 1, d, B, keys) == "streaming"
        assert form(192, 300, 1, d, F) == "streaming" and form(192, 512, 1, 64, F) == (1, 512)   # nearly two rounds of workgroups
    assert form(64, 128, 1, 128, B) == (2, 512) and form(64, 129, 1, 128, B) == (1, 512)   # one round of workgroups
    assert form(512, 4096, 8, 128, B) == (1, 512) and form(512, 4097, 8, 128, B) == "streaming"
    assert form(1024, 128, 1, 128, B) == (2, 512) and form(1024, 256, 1, 128, B) == "streaming"
    # few memories: KB of values of one workgroup's, of two
    own = P.BCT_MK_PER_SEQUENCE
    for M, n, G, d, dt, keys, last in ((640, 31, 1, 64, B, 0, 1), (640, 63, 1, 64, B, 0, 1), (320, 31, 1, 64, F, 0, 1),
                                       (384, 32, 1, 64, F, 0, 1), (768, 32, 1, 64, B, own, 1), (768, 16, 2, 64, B, 0, 1),
                                       (832, 40, 2, 64, B, 0, 1), (1024, 40, 2, 64, B, own, 1), (1024, 16, 3, 64, B, 0, 1),
                                       (512, 31, 1, 128, B, 0, 2), (640, 32, 1, 128, B, 0, 2), (640, 31, 2, 128, B, 0, 2),
                                       (256, 63, 1, 128, F, 0, 2)):
        assert form(M, n, G, d, dt, keys)[0] == last and form(M + 64, n, G, d, dt, keys) == "streaming", (M, n, G, d, dt, keys)
    # 64 to 128 memories, one round of long chains
    for M, n, G, d, keys in ((1088, 64, 1, 128, 0), (1088, 64, 2, 64, 0), (1216, 80, 1, 64, 0), (1600, 100, 2, 64, 0), (1536, 100, 1, 64, 0),
                             (1536, 128, 1, 64, 0), (1408, 64, 1, 64, own), (768, 64, 1, 128, own), (1664, 200, 1, 64, 0), (832, 200, 1, 128, 0),
                             (832, 600, 2, 128, 0), (1728, 600, 2, 64, 0), (256, 512, 1, 128, 0)):
        assert form(M, n, G, d, B, keys) != "streaming" and form(M + 64, n, G, d, B, keys) == "streaming", (M, n, G, d, keys)
    for n in (256, 304, 512):   # 1024 threads are alone on a compute unit: not somewhat more than a round of them
        assert form(576, n, 2, 128, B) == (1, 1024)
    assert form(576, 257, 2, 128, B) == form(576, 303, 2, 128, B) == "streaming" and form(512, 257, 2, 128, B) == (1, 512)
    # two workgroups of each of more than 128 memories
    for M, dt, G, first, end in ((576, B, 3, 192, 256), (576, B, 5, 192, 1024), (704, B, 5, 192, 256), (576, B, 8, 129, 1024),
                                 (320, F, 2, 208, 256), (320, F, 3, 192, 256), (320, F, 5, 129, 4096)):
        assert form(M, first, G, 128, dt)[0] == form(M, end, G, 128, dt)[0] == 2 and form(M, end + 1, G, 128, dt) == "streaming", (M, dt, G)
        if first > 129:
            assert form(M, first - 1, G, 128, dt) == "streaming", (M, dt, G)


def test_chunks_of_few_tokens(L):
    """One pass over keys and values: 32 rows (tokens x heads of a memory) always; 33 to 64 where a memory is one tile of 128 slots
    or there are 64 memories at most, if their operands and partial outputs fit where a chunk of 128 tokens keeps its values."""
    import itertools
    def one(B, H, G, d, M, T, dt=P.BCT_BF16):
        st, v = P.bct_plan_prefill(P.make_desc(M, B, H * G, H, d, dt, 0.1, 0.1, 0), T)
        assert st == P.BCT_OK
        return v
    for d, M, G, T in itertools.product((64, 128), (64, 128, 192, 256, 448, 1088, 4096, 65536), range(1, 9), (1, 7, 12, 15, 16, 31, 32, 33, 40, 45, 58, 64, 65)):
        rows, tiles = T * G, -(-M // 128)
        shares = -(-tiles // -(-tiles // 8))
        need = (2 * (2 if T > 32 else 1) + (2 if rows > 32 else 1)) * 64 * d + 8 * T * shares + (tiles > 1) * tiles * rows * (4 * d + 8)
        fits = need <= (128 + M) * 2 * d
        assert fits or rows > 32
        assert one(64, 1, G, d, M, T) == (rows <= 64 and fits), (d, M, G, T)
        assert one(65, 1, G, d, M, T) == (rows <= 64 and fits and (rows <= 32 or tiles == 1)), (d, M, G, T)
        assert one(1, 1, G, d, M, T, P.BCT_F32) == 0
    assert P.bct_plan_prefill(desc(), 0)[0] == P.BCT_ERR_INVALID_ARG
