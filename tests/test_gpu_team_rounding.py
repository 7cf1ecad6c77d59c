"""Splits that hover at the trivial point, where accepting a step hangs on the last
bit of the Gibbs energy: stable mixtures that the caller declares unstable.  The
forms that use teams (small batches, the tails of the fused and of the persistent
form) equal the plain form, which has none, bit for bit.  The batches each hold a
mixture whose path depends on the rounding of the energy's sum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import _capi, api, workloads  # noqa: E402
from parity import gpu_to_numpy  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,seed,n", [(4, 5805, 100_000), (5, 5904, 100_000),
                                       (7, 6103, 100_000), (8, 6207, 100_000),
                                       (9, 6304, 60_000), (10, 6406, 60_000),
                                       (11, 6504, 60_000), (12, 6605, 60_000)])
def test_forms_agree_at_the_trivial_point(nc, seed, n):
    print(f"case nc={nc} seed={seed} n={n}", flush=True)
    w = workloads.uniform_workload("near", seed, n, nc, 0.5, (200.0, 600.0), (1e5, 2e7))
    hint = np.ones(n, np.int8)

    def run(lo, hi, **kw):
        return gpu_to_numpy(api.flash(w.z[lo:hi], w.T[lo:hi], w.P[lo:hi], w.Tc, w.Pc, w.omega,
                                      w.kij, hint=hint[lo:hi], keep_factor=True, **kw))

    want = run(0, n, form=_capi.FORM_PLAIN)
    step = 10_000   # batches of this size take a team per mixture
    small = [run(lo, lo + step) for lo in range(0, n, step)]
    got = {"default": run(0, n), "fused": run(0, n, form=_capi.FORM_FUSED),
           "persistent": run(0, n, block=64, lanes_per_mixture=1),
           "small": {k: np.concatenate([s[k] for s in small]) for k in want}}
    for name, g in got.items():
        for k in ("label", "beta", "x", "y", "iters", "status", "flops", "tm", "factor"):
            assert np.array_equal(g[k], want[k], equal_nan=True), (name, k)
