"""The streaming step's matrix-core read of several query heads with 64 columns: edges of its 64-slot wavefronts and
128-slot workgroups, against the oracle."""
import pytest

import bct_synth as syn
from _util import make_pair, sub, to_dev, to_np
from test_gpu_parity import check_out, check_state_one_step

pytestmark = pytest.mark.gpu


# one wavefront of two with slots, a partial last workgroup, whole ones; statistics merged in the pass and by their own launch
@pytest.mark.parametrize("B,Hkv,G,M,seq", [(1, 1, 3, 64, 0), (3, 2, 4, 192, 0), (2, 3, 5, 1024, 1), (5, 1, 8, 2112, 0),
                                           (24, 43, 3, 2048, 0), (4, 64, 3, 2048, 0), (11, 8, 4, 4160, 1)])
def test_steps_from_a_common_state(B, Hkv, G, M, seq):
    import paper_2411_15785_amd as P
    from oracle import bct_ref as R
    w = syn.Workload("heads", 1, B, Hkv * G, Hkv, 64, M, "bf16", 3)
    few = [0, B - 1] if B > 8 else None
    ref, gpu, mk, mv, bs = make_pair(w, R.RefCache, P.BctCache, flags=seq | P.BCT_STEP_STREAMING, mv0=True, batch_subset=few)
    st, plan = P.bct_plan_query(gpu.desc)
    assert st == P.BCT_OK and plan["mv_workgroup"] == 128 and plan["mv_loads_per_lane"] == 8
    assert plan["normaliser_launch"] == (1 if B * Hkv * M > 16384 * 128 else 0)
    for t, (read, write) in enumerate(((True, True), (False, True), (True, False))):
        q, wq, wv = syn.make_step(w, t)
        q, wq, wv = q if read else None, wq if write else None, wv if write else None
        before = ref.values()
        whole = to_np(gpu.values_view(), "bf16").copy()
        whole[bs] = before
        gpu.set_values(to_dev(whole, "bf16"))
        o_ref = ref.decode_step(sub(q, bs), sub(wq, bs), sub(wv, bs))
        o = gpu.decode_step(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"))
        what = f"M={M} G={G} read={read} write={write}"
        if read:
            check_out(to_np(o, "bf16")[bs], o_ref, "bf16", what)
        check_state_one_step(to_np(gpu.values_view(), "bf16")[bs], ref.values(), "bf16", what, before=before)


# two, three and four tiles a workgroup, the last workgroup with one, with half a tile; statistics merged in the pass and by their
# own launch
@pytest.mark.parametrize("G,Hkv,M,seq,splits", [(3, 24, 15808, 0, 62), (4, 31, 10880, 1, 29), (8, 64, 3008, 0, 6),
                                               (8, 100, 1920, 0, 5)])
def test_more_slots_a_workgroup_where_the_static_scratch_ends(G, Hkv, M, seq, splits):
    import numpy as np
    import paper_2411_15785_amd as P
    from oracle import bct_ref as R
    import torch
    w = syn.Workload("heads_static", 1, 1, Hkv * G, Hkv, 64, M, "bf16", 3)
    ref, gpu, mk, mv, _ = make_pair(w, R.RefCache, P.BctCache, flags=seq | P.BCT_STEP_STREAMING, mv0=True)
    assert P.bct_plan_query(gpu.desc)[1]["mv_splits"] == splits
    for t, (read, write) in enumerate(((True, True), (False, True), (True, False))):
        q, wq, wv = syn.make_step(w, t)
        q, wq, wv = q if read else None, wq if write else None, wv if write else None
        before = ref.values()
        gpu.set_values(to_dev(before, "bf16"))
        o_ref = ref.decode_step(q, wq, wv)
        o = torch.empty((1, w.Hq, 64), dtype=torch.bfloat16, device="cuda:0") if read else None
        gpu.decode_step_static(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"), o)
        what = f"M={M} G={G} read={read} write={write}"
        if read:
            check_out(to_np(o, "bf16"), o_ref, "bf16", what)
        check_state_one_step(to_np(gpu.values_view(), "bf16"), ref.values(), "bf16", what, before=before)
        if read and write:
            state = gpu.values_view().clone()
            gpu.set_values(to_dev(before, "bf16"))
            again = gpu.decode_step(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"))
            assert torch.equal(o.view(torch.int16), again.view(torch.int16)) and torch.equal(state.view(torch.int16), gpu.values_view().view(torch.int16))
    assert np.array_equal(to_np(gpu.keys_view(), "bf16"), mk)


# streaming launches with 64 columns (one tile a workgroup, several); the whole step in one launch, 8 and 16 lanes to a slot row
@pytest.mark.parametrize("B,Hkv,G,d,M,whole", [(16, 4, 8, 64, 1088, 0), (1, 64, 8, 64, 3008, 0), (64, 4, 8, 64, 128, 1), (16, 8, 4, 128, 64, 2),
                                              (40, 4, 3, 128, 256, 1)])
def test_outputs_are_the_rounding_of_the_exact_read(B, Hkv, G, d, M, whole):
    """Weights keep their 24 bits on the matrix cores: the output differs from the rounding of the oracle's (64 bits, from the
    same stored values) where an fp32 sum would, in 1e-4 to 5e-4 of the elements (weights of 16 to 17 bits: 2e-3 and more).  An
    infinity in MV is read as one."""
    import numpy as np
    import paper_2411_15785_amd as P
    from oracle import bct_ref as R
    w = syn.Workload("heads_exact", 1, B, Hkv * G, Hkv, d, M, "bf16", 3)
    ref, gpu, mk, mv, _ = make_pair(w, R.RefCache, P.BctCache, mv0=True, flags=0 if whole else P.BCT_STEP_STREAMING)
    assert P.bct_plan_whole(gpu.desc)[1] == whole
    dev = lambda a: to_dev(a, "bf16")
    off = n = 0
    for t in range(3):
        q, wq, wv = syn.make_step(w, t)
        for c, a in ((ref, mv), (gpu, dev(mv))):
            c.set_values(a)
        o_ref, o = ref.decode_step(q, wq, wv), to_np(gpu.decode_step(dev(q), dev(wq), dev(wv)), "bf16")
        off, n = off + np.count_nonzero(o != o_ref), n + o.size
    assert n >= 30000 and off <= 1e-3 * n, f"{off} of {n}"
    inf = mv.copy()
    inf[0, 0, 5, 3], inf[B - 1, Hkv - 1, M - 1, d - 1], inf[0, 0, M // 2, 7] = 0x7F80, 0xFF80, 0x7F80
    for write in (True, False):
        for c, a in ((ref, inf), (gpu, dev(inf))):
            c.set_values(a)
        wq1, wv1 = (wq, wv) if write else (None, None)
        a, b = ref.decode_step(q, wq1, wv1), to_np(gpu.decode_step(dev(q), dev(wq1), dev(wv1)), "bf16")
        special = (a & 0x7F80) == 0x7F80
        assert np.count_nonzero(special) == 3 * G and np.array_equal(a[special], b[special])
        assert np.all((b[~special] & 0x7F80) != 0x7F80)
