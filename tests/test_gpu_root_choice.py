"""The choice between the liquid and the vapour root of the cubic, which the kernels take
from single-precision logarithms unless the two energies nearly tie: on the device, at
pressures next to the one where they tie, against the energies in extended precision."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import api  # noqa: E402

pytestmark = pytest.mark.gpu

LD = np.longdouble
DELTA = np.concatenate([s * np.logspace(-13, -1, 49) for s in (-1.0, 1.0)])


def _roots(A, B):
    """Smallest and largest real root of the cubic and whether it has three above B."""
    c1, c0 = A - B - B * B, -A * B
    p, q = c1 - LD(1) / 3, c0 + c1 / 3 - LD(2) / 27
    three = q * q / 4 + p * p * p / 27 < 0
    r = np.sqrt(np.where(three, -p / 3, LD(1)))
    th = np.arccos(np.clip(np.where(three, -q / 2 / r ** 3, LD(0)), -1, 1)) / 3
    out = []
    for j in (2, 0):
        Z = 2 * r * np.cos(th - 2 * LD(np.pi) * j / 3) + LD(1) / 3
        for _ in range(6):
            f = ((Z - 1) * Z + c1) * Z + c0
            fp = (3 * Z - 2) * Z + c1
            Z = np.where(three, Z - f / np.where(fp == 0, LD(1), fp), LD(1))
        out.append(Z)
    zl, zv = np.minimum(*out), np.maximum(*out)
    return zl, zv, three & (zl > B)


def _energy_gap(A, B):
    zl, zv, three = _roots(A, B)
    with np.errstate(invalid="ignore", divide="ignore"):
        g = lambda Z: Z - 1 - np.log(Z - B) - A / B * np.log1p(B / Z)
        return np.where(three, g(zv) - g(zl), LD(np.nan)), zl, zv


def test_root_choice_next_to_the_tie():
    rng = np.random.Generator(np.random.PCG64(8100))
    m = 4000
    Tc, Pc, om = np.array([304.0, 510.0]), np.array([4.1e6, 3.2e6]), np.array([0.2, 0.35])
    k = np.array([[0.0, 0.06], [0.06, 0.0]])
    x = rng.uniform(0.0, 1.0, m)
    c = np.stack([x, 1.0 - x], 1)
    T = rng.uniform(0.45, 0.97, m) * (c @ Tc)

    def AB(P, c, T):
        tr, pr = Tc / T[:, None], P[:, None] / Pc
        a = 1 + (0.480 + 1.574 * om - 0.176 * om ** 2) * (1 - np.sqrt(LD(1) / tr))
        s, b = np.abs(a) * tr * np.sqrt(LD(0.42748) * pr), LD(0.08664) * tr * pr
        psi = (s * c) @ (1 - k).astype(LD)
        return (s * c * psi).sum(1), (c * b).sum(1)

    # the last sign change of the gap along P, then bisection: vapour below, liquid above
    grid = np.exp(np.linspace(np.log(1e2), np.log(1.5e7), 240))
    gap = np.stack([_energy_gap(*AB(np.full(m, p, LD), c, T))[0] for p in grid])
    cross = (gap[:-1] < 0) & (gap[1:] >= 0)
    has = cross.any(0)
    i = len(grid) - 2 - np.argmax(cross[::-1], 0)
    lo, hi = grid[i].astype(LD), grid[i + 1].astype(LD)
    for _ in range(70):
        mid = np.sqrt(lo * hi)
        low = _energy_gap(*AB(mid, c, T))[0] < 0
        lo, hi = np.where(low, mid, lo), np.where(low, hi, mid)
    c, T, tie = c[has], T[has], hi[has].astype(np.float64)
    assert has.sum() > 1500
    P = (tie[:, None] * (1 + DELTA)).reshape(-1)
    c, T = np.repeat(c, len(DELTA), 0), np.repeat(T, len(DELTA))
    gap, zl, zv = _energy_gap(*AB(P.astype(LD), c, T))
    lnphi, Z, _ = api.eval_phase(c, T, P, Tc, Pc, om, k, derivs=False)
    Z = Z.cpu().numpy()
    vapour = np.abs(Z - zv) < np.abs(Z - zl)
    # 1e-13 of rounding in A, B and the energies themselves, 1000 units in the last place
    clear = np.isfinite(gap) & (np.abs(gap) > 1e-13) & (zv - zl > 1e-3)
    print("cases", clear.sum(), "within 1e-5 of a tie", (clear & (np.abs(gap) < 1e-5)).sum(),
          "vapour", (clear & vapour).sum(), flush=True)
    assert clear.sum() > 100_000 and (clear & (np.abs(gap) < 1e-5)).sum() > 20_000
    assert np.array_equal(vapour[clear], gap[clear] < 0)
    assert torch.isfinite(lnphi).all()
