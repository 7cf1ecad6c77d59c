"""The side streams of a ragged call, with HIP's stream calls replaced by ones that can
fail: a call goes on with the streams it could get and leaves no error behind, one under
capture takes none, and a join that cannot order the caller's stream waits on the host
and reports it."""
import os
import subprocess

import pytest

from host_items import runner


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    d = tmp_path_factory.mktemp("fork")
    os.makedirs(d / "hip")
    (d / "hip" / "hip_runtime_api.h").write_text("#pragma once\n")
    exe = str(d / "stream_fork")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(d),
                    "-I", os.path.join(runner.ROOT, "include"), "-I", runner.CSRC,
                    os.path.join(runner.HERE, "stream_fork.cpp"), "-o", exe, "-lpthread"],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return {line.split()[0]: [int(v) for v in line.split()[1:]] for line in out.splitlines()}


EHIP = 4


@pytest.mark.parametrize("case,want", [
    # streams, error left, join's code, waits of the caller's stream, synchronisations
    ("all", [4, 0, 0, 3, 0]), ("again", [4, 0, 0, 3, 0]), ("two", [2, 0, 0, 1, 0]),
    ("one", [1, 0, 0, 0, 0]), ("capture", [1, 0, 0, 0, 0]), ("second_wait", [2, 0, 0, 1, 0]),
    ("first_wait", [1, 0, 0, 0, 0]), ("join", [4, 0, EHIP, 0, 3]),
    ("create", [1, 0, 0, 0, 0]), ("create_again", [1, 0, 0, 0, 0]), ("after", [4, 0, 0, 3, 0])])
def test_fork_and_join(report, case, want):
    assert report[case] == want
