"""Splits that spend a full budget of steps, restart and spend another: the plain form
steps them to their end as the other forms do."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [3, 4, 7])
def test_plain_form_finishes_restarted_splits(nc):
    print(f"case nc={nc}", flush=True)
    w = workloads.uniform_workload("restart", 7300 + nc, 40_000, nc, 0.5, (200.0, 600.0),
                                   (1e5, 2e7))
    args = (w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij)
    kw = dict(max_ss=2, dem_every=2, tol_sa_ss=1e-16, tol_sa_tr=1e-16, tol_split_tr=1e-16,
              max_tr_sa=40, max_tr_split=60)
    a = gpu_to_numpy(api.flash(*args, form=_capi.FORM_PLAIN, **kw))
    b = gpu_to_numpy(api.flash(*args, block=64, lanes_per_mixture=1, lanes_ss=1, **kw))
    for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm"):
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    assert (b["iters"][:, 6] > 96).any()   # more trust-region steps than one budget
