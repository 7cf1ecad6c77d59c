"""The groups of a ragged batch run on several streams, in rounds where the
workspace does not hold them side by side.  Every component count at batch
sizes whose groups need more than one round or are single mixtures, calls on
a stream of the caller's own whose inputs are written on it just before, and
calls from several threads at once: each equals, bit for bit, the uniform
flash of each group."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2205_03090_amd import api, workloads  # noqa: E402

pytestmark = pytest.mark.gpu

FIELDS = ("label", "beta", "iters", "status", "flops", "tm")


def _call(w, stream=None):
    dev = torch.device("cuda", 0)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev)
    return api.flash_ragged(t(w.z), t(w.T), t(w.P), w.nc_of, w.off, w.koff, t(w.Tc), t(w.Pc),
                            t(w.omega), t(w.kij), stream=stream)


def _expect(w):
    out = {}
    for nc in sorted(set(w.nc_of.tolist())):
        idx, g = w.group(nc)
        out[nc] = (idx, api.flash(g.z, g.T, g.P, g.Tc, g.Pc, g.omega, g.kij))
    torch.cuda.synchronize()
    return out


def _check(w, r, want):
    for nc, (idx, u) in want.items():
        for k in FIELDS:
            assert np.array_equal(getattr(r, k).cpu().numpy()[idx],
                                  getattr(u, k).cpu().numpy(), equal_nan=True), (nc, k)
        rows = w.off[idx][:, None] + np.arange(nc)[None, :]
        for k in ("x", "y"):
            assert np.array_equal(getattr(r, k).cpu().numpy()[rows],
                                  getattr(u, k).cpu().numpy()), (nc, k)


@pytest.mark.parametrize("n", [1, 5, 40, 700, 6000])
def test_every_component_count(n):
    print(f"case n={n}", flush=True)
    w = workloads.ragged_workload("rs", 6100 + n, n, nc_set=tuple(range(2, 21)))
    _check(w, _call(w), _expect(w))


def test_caller_stream_orders_the_side_streams():
    w = workloads.ragged_workload("rs", 6200, 3000, nc_set=(2, 5, 9, 16, 20))
    want = _expect(w)
    s = torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(s):
            r = _call(w, s)                       # inputs copied on s, then the call
            tail = [getattr(r, k).clone() for k in ("label", "beta")]   # ordered after it
        s.synchronize()
        _check(w, r, want)
        assert torch.equal(tail[0], r.label) and torch.equal(tail[1], r.beta)


def test_threads():
    ws = [workloads.ragged_workload("rs", 6300 + k, 1500, nc_set=(3, 8, 12, 20))
          for k in range(6)]
    wants = [_expect(w) for w in ws]
    got, errors = [None] * len(ws), []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(3):
                    got[k] = _call(ws[k], s)
            s.synchronize()
        except Exception as e:   # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(ws))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    for w, r, want in zip(ws, got, wants):
        _check(w, r, want)
