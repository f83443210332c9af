"""The tuner against handles left alone: the untuned shape, which cuts the z
range of small launches, is one of its candidates."""
import json

import numpy as np
import pytest

from paper_2609_13115_amd import workloads, xls

pytestmark = pytest.mark.gpu


# Whole boxes take about four times as long here (one wave of workgroups for a
# cell of 24^3 points with 20 columns); the filter is most of an iteration.
@pytest.mark.parametrize("prec", [xls.XLS_PREC_FP64, xls.XLS_PREC_FP32])
def test_a_tuned_small_batch_is_not_slower(prec, tmp_path):
    sds = [workloads.small_periodic(n=24, ns=20, index=3)]
    params = [xls.chefsi_params(60, 6, xls.XLS_BOUNDS_LANCZOS)]
    path = str(tmp_path / "tune.json")
    ms = []
    for tuned in (False, True):
        print(f"[case] tuned small batch prec={prec} tuned={tuned}", flush=True)
        with xls.Batch(sds, filter_prec=prec) as b:
            if tuned:
                b.xls_batch_tune(path)
            t = []
            for _ in range(3):
                b.xls_batch_chefsi(params)
                t.append(b.xls_batch_stats()["last_iter_ms"])
            ms.append(min(t))
    shape = json.load(open(path))[xls.tune_keys(sds[0], prec)[0]]
    print(f"[tune] untuned {ms[0]:.3f} ms, tuned {ms[1]:.3f} ms, shape {shape}", flush=True)
    assert ms[1] <= 1.25 * ms[0]


# An entry of a file whose candidates did not have the untuned shape (its key
# says so) is timed again; an entry that names the untuned shape restores it on a
# handle that was tuned.
def test_cache_entries_of_earlier_candidates_and_the_untuned_shape(tmp_path):
    print("[case] tune cache", flush=True)
    sd = workloads.small_dirichlet(ns=10, index=1, shape=(13, 9, 20), h=0.6)
    skey, gkey = xls.tune_keys(sd, xls.XLS_PREC_FP32)
    old = {"f32_nx13_ny16_nz24_d_na64": [512, 16, 2], "gemm_f32_nd32768_ns32": [8, 1, 1]}
    path = tmp_path / "tune.json"
    path.write_text("{\n" + ",\n".join(f'  "{k}": {v}' for k, v in old.items()) + "\n}\n")
    with xls.Batch([sd], filter_prec=xls.XLS_PREC_FP32) as b:
        assert b.xls_batch_tune(str(path))[0] == 2
    got = json.load(open(path))
    assert set(got) == set(old) | {skey, gkey} and all(got[k] == old[k] for k in old)
    path.write_text("{\n" + f'  "{skey}": [512, 0, 1],\n  "{gkey}": [0, 0, 0]\n' + "}\n")
    params = [xls.chefsi_params(7, 4, xls.XLS_BOUNDS_LANCZOS)]
    with xls.Batch([sd], filter_prec=xls.XLS_PREC_FP32) as b:
        b.xls_batch_subdomain(0).xls_subdomain_tune(xls.XLS_PREC_FP32, 256, 2, 4, 1)
        assert b.xls_batch_tune(str(path))[0] == 0
        b.xls_batch_chefsi(params)
        b.xls_batch_subdomain(0).xls_subdomain_tune(xls.XLS_PREC_FP32, 0, 0, 0, 0)
        b.xls_batch_chefsi(params)
        assert b.xls_batch_stats()["captures"] == 1
        resid = b.xls_batch_subdomain(0).xls_subdomain_residual(np.zeros(10))
    assert np.all(np.isfinite(resid))
