"""The batch sizes at which the default form changes, from a team of lanes per mixture
to a lane pair and from one launch to a launch per stage (csrc/form_limits.hpp), and
sizes whose wavefronts hold a team in every slot: the flash and the stability analysis
on both sides of each limit equal the plain form, which has neither teams nor pairs,
bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, autotune, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu

TEAM, FUSED = autotune.form_limits()


def _workload(nc, per, n):
    make = workloads.per_mixture_workload_vec if per else workloads.uniform_workload
    return make("limit", 5600 + nc, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7))


def _check(nc, per, n, stability):
    print(f"case nc={nc} per={per} n={n} stability={stability}", flush=True)
    w = _workload(nc, per, n)
    args = (w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij)
    if stability:
        a, b = api.stability(*args), api.stability(*args, form=_capi.FORM_PLAIN)
        for k in ("label", "iters", "status", "flops", "tm"):
            assert np.array_equal(getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy(),
                                  equal_nan=True), k
        return
    a = gpu_to_numpy(api.flash(*args, keep_factor=True))
    b = gpu_to_numpy(api.flash(*args, keep_factor=True, form=_capi.FORM_PLAIN))
    for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm", "factor"):
        assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("stability", [False, True])
@pytest.mark.parametrize("nc,per", [(2, True), (4, False), (5, False), (8, True), (12, False)])
def test_team_limit(nc, per, stability):
    limit = TEAM[int(stability)][nc]
    for n in (limit, limit + 1):
        _check(nc, per, n, stability)


@pytest.mark.parametrize("nc,per,n", [(2, False, 9001), (3, True, 7999), (4, True, 19_999),
                                      (5, True, 3501), (7, False, 4097), (8, False, 9999),
                                      (9, False, 3073), (10, True, 7003), (11, False, 5002),
                                      (11, True, 3998), (12, True, 9_998)])
def test_every_team_slot(nc, per, n):
    _check(nc, per, n, False)


@pytest.mark.parametrize("stability", [False, True])
@pytest.mark.parametrize("nc,per", [(4, False), (8, False), (9, True)])
def test_fused_limit(nc, per, stability):
    limit = FUSED[int(stability)][nc]
    for n in (limit, limit + 1):
        _check(nc, per, n, stability)


@pytest.mark.parametrize("nc,per", [(12, True), (13, False), (20, False)])
def test_fused_limit_above_the_lane_forms(nc, per):
    """From nc 12 (own sets) or 13 on, the staged form's trust regions may run in lane
    groups, whose sums have another order: only the fused side is compared bit for bit."""
    _check(nc, per, FUSED[0][nc], False)
