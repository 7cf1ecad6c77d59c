"""The component counts with teams at the end of the split trust region that
test_gpu_tail.py does not compare: every output equals the plain form's, which has no
teams, bit for bit, with shared and own sets."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(nc, per, n, **shape):
    print(f"case nc={nc} per={per} n={n} {shape}", flush=True)
    make = workloads.per_mixture_workload_vec if per else workloads.uniform_workload
    w = make("tail", 5500 + nc, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7))
    args = (w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij)
    a = gpu_to_numpy(api.flash(*args, keep_factor=True, **shape))
    b = gpu_to_numpy(api.flash(*args, keep_factor=True, form=_capi.FORM_PLAIN))
    for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm", "factor"):
        if k in a or k in b:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("nc,per", [(2, False), (2, True), (3, False), (3, True), (7, True)])
@pytest.mark.parametrize("n", [1, 70, 3001, 160_003])
def test_persistent_tail(nc, per, n):
    _check(nc, per, n, block=64, lanes_per_mixture=1)


@pytest.mark.parametrize("nc,per", [(2, True), (3, False), (3, True), (6, False), (7, False),
                                    (7, True), (9, True), (10, False), (10, True), (11, False),
                                    (11, True), (12, False)])
@pytest.mark.parametrize("n", [1, 33, 3001, 40_003])
def test_fused_tail(nc, per, n):
    _check(nc, per, n, form=_capi.FORM_FUSED)
