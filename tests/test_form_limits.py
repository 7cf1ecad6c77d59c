"""The autotuner's account of the default form against the limits that the library
compiles in (csrc/form_limits.hpp) and that the header states."""
import os
import re

import pytest

from paper_2205_03090_amd import autotune

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TEAM, FUSED = autotune.form_limits()


@pytest.mark.parametrize("nc", range(2, 21))
@pytest.mark.parametrize("stability", [False, True])
def test_default_form_follows_the_limits(nc, stability):
    team, fused = TEAM[int(stability)][nc], FUSED[int(stability)][nc]
    assert 0 <= team < fused
    form = lambda n: autotune.default_form(nc, n, stability)
    if team:
        assert form(1) == form(team) == "team"
    assert form(team + 1) == form(fused) == "fused"
    assert form(fused + 1) == "persistent"
    if not stability:
        assert autotune.fused_default(nc, fused) and not autotune.fused_default(nc, fused + 1)


def test_header_states_the_limits():
    text = open(os.path.join(ROOT, "include", "ptflash.h")).read()
    text = re.sub(r"[\s*]+", " ", text[text.index("#define PTFLASH_FORM_PERSISTENT"):
                                      text.index("#define PTFLASH_FORM_PLAIN")])
    m = re.search(r"n <= (\d+) \(nc <= 4\), (\d+) \(nc <= 8\), (\d+) \(nc = 9\), (\d+) \(nc = 10\), "
                  r"(\d+) \(nc <= 12\) or n nc <= (\d+)", text)
    f4, f8, f9, f10, f12, prod = (int(v) for v in m.groups())
    for nc in range(2, 21):
        want = f4 if nc <= 4 else f8 if nc <= 8 else f9 if nc == 9 else f10 if nc == 10 \
            else f12 if nc <= 12 else prod // nc
        assert FUSED[0][nc] == want, nc
    m = re.search(r"n <= (\d+) at nc <= 4, n <= (\d+) up to nc = 12", text)
    assert [TEAM[0][nc] for nc in (4, 5, 12, 13)] == [int(m[1]), int(m[2]), int(m[2]), 0]
    m = re.search(r"up to (\d+) at nc = 9 and 10, and with teams for n <= (\d+) \(nc <= 4\) and "
                  r"(\d+) \(nc <= 12\)", text)
    assert [FUSED[1][9], FUSED[1][10], TEAM[1][4], TEAM[1][12]] == [int(m[1])] * 2 + \
        [int(m[2]), int(m[3])]
