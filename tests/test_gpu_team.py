"""The smallest batches run with a team of lanes per mixture: every output
equals the lane-pair fused form's and the persistent form's bit for bit.
Component counts on both sides of the team's widths (4 and 8 members per
phase), of one, two and three components per member, and of the last count
with teams; batch sizes of one mixture, a partly filled wavefront, the step
from one to two mixtures per wavefront, and the limits of the form (one
mixture past them the lane pair runs)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu

FIELDS = ("label", "beta", "x", "y", "iters", "status", "flops", "tm", "factor")


def _same(a, b):
    for k in FIELDS:
        if k in a or k in b:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


def _args(w):
    return (w.z, w.T, w.P, w.Tc, w.Pc, w.omega, w.kij)


@pytest.mark.parametrize("nc,per", [(2, False), (3, True), (4, False), (5, True), (8, False),
                                    (9, True), (12, False)])
@pytest.mark.parametrize("n", [1, 13, 1024, 1025, 3001])
def test_team_equals_the_other_forms(nc, per, n):
    print(f"case nc={nc} per={per} n={n}", flush=True)
    w = workloads.uniform_workload("team", 5100 + nc, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7),
                                   per_mixture=per)
    team = gpu_to_numpy(api.flash(*_args(w), keep_factor=True))
    _same(team, gpu_to_numpy(api.flash(*_args(w), keep_factor=True, form=_capi.FORM_FUSED)))
    _same(team, gpu_to_numpy(api.flash(*_args(w), keep_factor=True, block=64,
                                       lanes_per_mixture=1)))


@pytest.mark.parametrize("nc,limit", [(4, 24000), (12, 12000)])
def test_team_limit(nc, limit):
    for n in (limit, limit + 1):
        print(f"case nc={nc} n={n}", flush=True)
        w = workloads.uniform_workload("team", 5200 + nc, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7))
        _same(gpu_to_numpy(api.flash(*_args(w))),
              gpu_to_numpy(api.flash(*_args(w), form=_capi.FORM_FUSED)))


def test_team_warm_start_stability_and_invalid_rows():
    """Hints, an initial K, rows the input checks refuse, and the stability
    analysis alone take the same paths as in the lane-pair form."""
    w = workloads.nc8_workload(n=1500, seed=91)
    z, P = w.z.copy(), w.P.copy()
    z[7, 2], P[40] = 0.0, np.nan
    rng = np.random.Generator(np.random.PCG64(92))
    hint = rng.integers(-1, 2, w.n).astype(np.int8)
    lnk0 = np.log(w.Pc / w.P[:, None]) + 5.373 * (1 + w.omega) * (1 - w.Tc / w.T[:, None])
    lnk0 += 0.05 * rng.standard_normal(lnk0.shape)
    args = (z, w.T, P, w.Tc, w.Pc, w.omega, w.kij)
    for kw in (dict(), dict(hint=hint), dict(lnk0=lnk0), dict(hint=hint, lnk0=lnk0)):
        _same(gpu_to_numpy(api.flash(*args, **kw)),
              gpu_to_numpy(api.flash(*args, form=_capi.FORM_FUSED, **kw)))
        a, b = api.stability(*args, **kw), api.stability(*args, form=_capi.FORM_FUSED, **kw)
        for k in ("label", "iters", "status", "flops", "tm"):
            assert np.array_equal(getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy(),
                                  equal_nan=True), k
