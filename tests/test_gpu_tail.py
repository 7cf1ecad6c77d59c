"""The last items of the split trust region's wavefronts, in the persistent and
in the fused form, are finished by teams of lanes: every output equals the
plain form's (one launch per step, no teams) bit for bit.  Component counts on
both sides of the ranges with teams; batches whose wavefronts start with fewer
items than teams, with lanes past the last mixture, with all lanes live, and
with several items per lane."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(nc, per, n, **shape):
    make = workloads.per_mixture_workload_vec if per else workloads.uniform_workload
    w = make("tail", 5300 + nc, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7))
    args = (w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij)
    a = gpu_to_numpy(api.flash(*args, keep_factor=True, **shape))
    b = gpu_to_numpy(api.flash(*args, keep_factor=True, form=_capi.FORM_PLAIN))
    for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm", "factor"):
        if k in a or k in b:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("nc,per", [(4, False), (5, False), (6, True), (7, False), (8, False),
                                    (8, True), (9, False)])
@pytest.mark.parametrize("n", [1, 70, 3001, 160003])
@pytest.mark.parametrize("block", [64, 256])
def test_tail_equals_the_plain_form(nc, per, n, block):
    print(f"case nc={nc} per={per} n={n} block={block}", flush=True)
    _check(nc, per, n, block=block, lanes_per_mixture=1)


@pytest.mark.parametrize("nc,per", [(2, False), (4, True), (5, False), (8, True), (9, False),
                                    (12, True), (13, False)])
@pytest.mark.parametrize("n", [1, 31, 33, 3001])
@pytest.mark.parametrize("block", [64, 256])
def test_fused_tail_equals_the_plain_form(nc, per, n, block):
    print(f"case nc={nc} per={per} n={n} block={block}", flush=True)
    _check(nc, per, n, block=block, form=_capi.FORM_FUSED)
