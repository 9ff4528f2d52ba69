"""Large grids whose workgroups take two tiles of slots, one after the other: an even and an odd number of tiles and a memory that
is one workgroup's, in steps that read and write, only write (one tile a workgroup again) and only read, against the oracle."""
import numpy as np
import pytest

import bct_synth as syn
from _util import make_pair, sub, to_dev, to_np
from test_gpu_parity import check_out, check_state_one_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,G,M,splits", [(1020, 3, 4, 1280, 10), (1000, 3, 8, 1344, 11), (2000, 8, 8, 128, 1),
                                              (1000, 3, 4, 1344, 21), (2001, 8, 8, 192, 3)])
def test_steps(B, Hkv, G, M, splits):
    import paper_2411_15785_amd as P
    from oracle import bct_ref as R
    import torch
    w = syn.Workload("tiles", 1, B, Hkv * G, Hkv, 128, M, "bf16", 5)
    bs = [0, B // 2, B - 1]
    ref, gpu, mk, _, _ = make_pair(w, R.RefCache, P.BctCache, batch_subset=bs)
    gpu.randomize_values(7, 1.0)
    assert P.bct_plan_rescores(gpu.desc) == (P.BCT_OK, 1) and P.bct_plan_query(gpu.desc)[1]["mv_splits"] == splits
    for t, (read, write) in enumerate(((True, True), (False, True), (True, False))):
        q, wq, wv = syn.make_step(w, t)
        q, wq, wv = q if read else None, wq if write else None, wv if write else None
        before = to_np(gpu.values_view()[bs], "bf16")
        whole = gpu.values_view().clone()
        ref.set_values(before)
        o_ref = ref.decode_step(sub(q, bs), sub(wq, bs), sub(wv, bs))
        o = gpu.decode_step(to_dev(q, "bf16"), to_dev(wq, "bf16"), to_dev(wv, "bf16"))
        what = f"M={M} G={G} read={read} write={write}"
        got = gpu.values_view()
        if read:
            check_out(to_np(o[bs], "bf16"), o_ref, "bf16", what)
        if write:
            check_state_one_step(to_np(got[bs], "bf16"), ref.values(), "bf16", what, before=before)
            assert bool((got != whole).flatten(2).any(dim=2).all())   # every memory was written
        else:
            assert torch.equal(got.view(torch.int16), whole.view(torch.int16))
    assert np.array_equal(to_np(gpu.keys_view(), "bf16"), mk)


@pytest.mark.parametrize("B,Hkv,G,M", [(1020, 3, 4, 1280), (1000, 3, 8, 1344)])
def test_steps_with_keys_of_each_sequence(B, Hkv, G, M):
    """Grids as large, of keys that cannot be scored again from a shared table: one tile a workgroup, all slots are taken."""
    import paper_2411_15785_amd as P
    from oracle import bct_ref as R
    import torch
    w = syn.Workload("tiles_own_keys", 1, B, Hkv * G, Hkv, 128, M, "bf16", 5)
    bs = [0, B - 1]
    gpu = P.BctCache(M, B, Hkv * G, Hkv, 128, torch.bfloat16, w.scale, w.scale, P.BCT_MK_PER_SEQUENCE)
    ref = R.RefCache(M, len(bs), Hkv * G, Hkv, 128, "bf16", w.scale, w.scale, P.BCT_MK_PER_SEQUENCE)
    gpu.set_keys(torch.randn((B, Hkv, M, 128), generator=torch.Generator("cuda:0").manual_seed(3), device="cuda:0",
                             dtype=torch.bfloat16))
    gpu.randomize_values(7, 1.0)
    assert P.bct_plan_rescores(gpu.desc) == (P.BCT_OK, 0) and P.bct_plan_query(gpu.desc)[1]["mv_splits"] == M // 64
    for t, (read, keyed) in enumerate(((True, False), (False, False), (True, True))):
        q, wq, wv = syn.make_step(w, t)
        wk = np.roll(wq, 1, axis=-1) if keyed else None
        q = q if read else None
        before = to_np(gpu.values_view()[bs], "bf16")
        keys = to_np(gpu.keys_view()[bs], "bf16")
        ref.set_keys(keys)
        ref.set_values(before)
        what = f"M={M} G={G} read={read} keyed={keyed}"
        dev = [to_dev(a, "bf16") for a in (q, wq, wv, wk)]
        if keyed:
            o = gpu.decode_step_keyed(*dev)
            o_ref = ref.decode_step_keyed(sub(q, bs), sub(wq, bs), sub(wv, bs), sub(wk, bs))
            check_state_one_step(to_np(gpu.keys_view()[bs], "bf16"), ref.keys(), "bf16", what + " keys", before=keys)
        else:
            o = gpu.decode_step(*dev[:3])
            o_ref = ref.decode_step(sub(q, bs), sub(wq, bs), sub(wv, bs))
        if read:
            check_out(to_np(o[bs], "bf16"), o_ref, "bf16", what)
        check_state_one_step(to_np(gpu.values_view()[bs], "bf16"), ref.values(), "bf16", what, before=before)


# 64 columns, M an odd multiple of 64, much of it: the vector-ALU pass of 512 slots a workgroup, the last one partly used
@pytest.mark.parametrize("B,Hkv,G,M,seq", [(110, 8, 3, 7104, 0), (110, 8, 3, 7104, 1), (83, 8, 4, 14144, 0)])
def test_odd_memories_of_64_columns(B, Hkv, G, M, seq):
    import paper_2411_15785_amd as P
    from oracle import bct_ref as R
    import torch
    w = syn.Workload("odd64", 1, B, Hkv * G, Hkv, 64, M, "bf16", 5)
    bs = [0, B - 1]
    gpu = P.BctCache(M, B, Hkv * G, Hkv, 64, torch.bfloat16, w.scale, w.scale, seq)
    ref = R.RefCache(M, len(bs), Hkv * G, Hkv, 64, "bf16", w.scale, w.scale, seq)
    st, plan = P.bct_plan_query(gpu.desc)
    assert plan["mv_workgroup"] == 512 and plan["mv_splits"] == -(-M // 512)
    gpu.set_keys(torch.randn(gpu.keys_shape, generator=torch.Generator("cuda:0").manual_seed(3), device="cuda:0", dtype=torch.bfloat16))
    gpu.randomize_values(7, 1.0)
    for t, (read, write, keyed) in enumerate(((True, True, False), (False, True, False), (True, False, False), (True, True, bool(seq)))):
        q, wq, wv = syn.make_step(w, t)
        wk = np.roll(wq, 1, axis=-1) if keyed else None
        q, wq, wv = q if read else None, wq if write else None, wv if write else None
        before = to_np(gpu.values_view()[bs], "bf16")
        keys = to_np(gpu.keys_view()[bs] if seq else gpu.keys_view(), "bf16")
        ref.set_keys(keys)
        ref.set_values(before)
        what = f"M={M} G={G} read={read} write={write} keyed={keyed}"
        dev = [to_dev(a, "bf16") for a in (q, wq, wv, wk)]
        if keyed:
            o = gpu.decode_step_keyed(*dev)
            o_ref = ref.decode_step_keyed(sub(q, bs), sub(wq, bs), sub(wv, bs), sub(wk, bs))
            check_state_one_step(to_np(gpu.keys_view()[bs], "bf16"), ref.keys(), "bf16", what + " keys", before=keys)
        else:
            o = gpu.decode_step(*dev[:3])
            o_ref = ref.decode_step(sub(q, bs), sub(wq, bs), sub(wv, bs))
        if read:
            check_out(to_np(o[bs], "bf16"), o_ref, "bf16", what)
        check_state_one_step(to_np(gpu.values_view()[bs], "bf16"), ref.values(), "bf16", what, before=before)
