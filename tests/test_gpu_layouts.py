"""One component set for the batch and the same set repeated for every mixture are
the same problem: outputs and factors agree bit for bit, in the default form and
with one launch per step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [2, 3, 5, 8, 12])
@pytest.mark.parametrize("form", [_capi.FORM_PERSISTENT, _capi.FORM_PLAIN])
def test_shared_set_equals_repeated_set(nc, form):
    print(f"case nc={nc} form={form}", flush=True)
    n = 30_000
    w = workloads.uniform_workload("layout", 7200 + nc, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7))
    rep = [np.ascontiguousarray(np.broadcast_to(a, (n,) + a.shape))
           for a in (w.Tc, w.Pc, w.omega, w.kij)]
    a = gpu_to_numpy(api.flash(w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij, keep_factor=True,
                               form=form))
    b = gpu_to_numpy(api.flash(w.z, w.T, w.P, *rep, keep_factor=True, form=form))
    for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm", "factor"):
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    assert (a["label"] == 1).mean() > 0.05
