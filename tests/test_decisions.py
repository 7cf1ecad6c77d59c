"""Decisions that the kernels settle without the logarithm, exponential or
quotient they are defined by (gibbs_order, ss_far, trivial_split, cut_step),
compiled for the host and compared with the definitions: on random inputs, on
inputs next to the threshold, and on zeros, infinities and NaN.  A shortcut
may leave a case open; it may never contradict."""
import os
import subprocess

import pytest

from host_items import runner


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("decisions") / "decisions")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off",
                    "-I", os.path.join(runner.HERE, "stub"),
                    "-I", os.path.join(runner.ROOT, "include"), "-I", runner.CSRC,
                    "-DPTF_MAX_NC=20", os.path.join(runner.HERE, "decisions.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return {line.split()[0]: [int(v) for v in line.split()[1:]] for line in out.splitlines()}


@pytest.mark.parametrize("name", ["gibbs_order", "ss_far", "trivial_split", "cut_step"])
def test_shortcut_never_contradicts_its_definition(report, name):
    cases, contradictions, settled = report[name]
    print(name, report[name])
    assert cases > 500_000 and contradictions == 0
    assert 0 < settled < cases   # both outcomes were met
