"""The lanes of a group share one mixture and exchange values at every step, while
each holds the mixture's scalars equal up to the last bit only.  The group's code
compiled for the host, one context per lane, with such a difference put in: the
lanes take the same path through every stage, at the default tolerances and at
tolerances of rounding size, where most decisions are between values that agree up
to the difference."""
import os
import subprocess

import pytest

from host_items import runner


@pytest.mark.parametrize("nc", [8, 12, 17])
def test_lanes_of_a_group_never_part(nc, tmp_path):
    exe = str(tmp_path / "group_lanes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off",
                    "-I", os.path.join(runner.HERE, "stub"),
                    "-I", os.path.join(runner.ROOT, "include"), "-I", runner.CSRC,
                    "-DPTF_MAX_NC=20", f"-DHOST_NC={nc}",
                    os.path.join(runner.HERE, "group_lanes.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    for n, tol in ((60, 1e-8), (40, 1e-16)):
        out = subprocess.run([exe, str(n), str(tol)], check=True, capture_output=True, text=True,
                             timeout=300).stdout
        items, steps, decisions, mixed, parted = (int(v) for v in out.split())
        print(nc, tol, out.strip())
        assert items > n and steps > 5 * items and decisions > 5 * steps
        assert parted == 0
    assert mixed > 0   # the lanes alone would have parted
