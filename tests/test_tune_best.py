"""The tuner's comparison of trial times (CPU): the candidate that is taken is the
one whose time is compared and stored."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(GXX is None, reason="g++ not available")


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tune") / "tune_best")
    subprocess.run([GXX, "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2112_03851_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "tune_best.cpp"), "-o", exe], check=True)

    def run(*trials):
        out = subprocess.run([exe, *(str(v) for t in trials for v in t)], capture_output=True, text=True, check=True)
        c, cms, s, sms, form = out.stdout.split()
        return int(c), float(cms), int(s), float(sms), form

    return run


@pytest.mark.parametrize("trials,taken", [
    ([(3, 1.0), (4, 1.02)], (3, 1.0)),      # larger, later and slower by 2 %
    ([(3, 1.0), (4, 0.995)], (3, 1.0)),     # near-equal: the earliest
    ([(3, 1.0), (4, 0.98)], (4, 0.98)),
    ([(2, float("inf")), (4, 2.0)], (4, 2.0))])
def test_a_slower_team_is_not_taken(pick, trials, taken):
    assert pick(*(("c", t, ms) for t, ms in trials))[:2] == taken


def test_forms_are_compared_by_the_times_of_what_would_run(pick):
    trials = [("c", 3, 1.0), ("c", 4, 1.02)]
    assert pick(*trials, ("s", 8, 0.985))[4] == "streaming"
    assert pick(*trials, ("s", 8, 0.995))[4] == "chip"
    assert pick(("s", 8, 0.995))[4] == "streaming"
    assert pick(("c", 3, 1.0))[4] == "chip"
    assert pick()[4] == "streaming"   # (nothing usable: the set-up shape stays)
