"""Lane groups at tolerances of rounding size, where most decisions are between
values that agree up to the last bit: every item ends, a mixture's outputs do not
depend on the launch shape, and the splits are valid and those of the default
tolerances.  (The lanes' common path is shown on the CPU in test_group_lanes.py.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import api, workloads  # noqa: E402
from parity import gpu_to_numpy, invariants  # noqa: E402

pytestmark = pytest.mark.gpu

TIGHT = dict(tol_sa_ss=1e-16, tol_sa_tr=1e-16, tol_split_ss=1e-16, tol_split_tr=1e-16, max_ss=30)


@pytest.mark.parametrize("nc,lanes,ss,per", [(8, 16, 16, False), (12, 16, 16, True),
                                             (16, 16, 1, False), (17, 32, 32, False),
                                             (20, 32, 32, True)])
def test_tight_tolerances(nc, lanes, ss, per):
    print(f"case nc={nc} lanes={lanes} ss={ss} per={per}", flush=True)
    w = workloads.uniform_workload("tight", 7100 + nc, 3000, nc, 0.5, (200.0, 600.0), (1e5, 2e7),
                                   per_mixture=per)
    args = (w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij)
    kw = dict(lanes_per_mixture=lanes, lanes_ss=ss)
    a = gpu_to_numpy(api.flash(*args, **kw, **TIGHT))
    b = gpu_to_numpy(api.flash(*args, **kw, **TIGHT, grid=7, block=64))
    for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm"):
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    inv = invariants(w, a)
    assert inv["mass_balance"] < 1e-13 and inv["sum_x"] < 1e-13 and inv["sum_y"] < 1e-13
    assert inv["single_ok"] and inv["beta_in_range"] and inv["labels_valid"]
    d = gpu_to_numpy(api.flash(*args))
    assert (a["label"] != d["label"]).mean() <= 0.01
    # two splits, both converged at the default criteria or better
    two = (a["label"] == 1) & (d["label"] == 1) & ((d["status"].astype(np.int64) & 0x20) == 0)
    assert two.sum() > 100
    assert np.quantile(np.abs(a["beta"][two] - d["beta"][two]), 0.99) < 1e-8
