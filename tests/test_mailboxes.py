"""The mailboxes between the members of a team in the on-chip fused CG (CPU): the
numbering rules of csrc/sos_mail.h under every order of the members' steps."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_03851_amd", "csrc")
GXX = shutil.which("g++")

pytestmark = pytest.mark.skipif(GXX is None, reason="g++ not available")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("mail") / "mail_model")
    subprocess.run([GXX, "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "mail_model.cpp"), "-o", exe], check=True)
    run = lambda members, counts_skipped, first, jobs: subprocess.run(
        [exe, str(members), str(int(counts_skipped)), str(first), *map(str, jobs)], capture_output=True, text=True,
        timeout=100)
    run.numbers = lambda *a: tuple(map(int, subprocess.run([exe, "numbers", *map(str, a)], capture_output=True,
                                                           text=True, check=True).stdout.split()))
    return run


@pytest.mark.parametrize("members,jobs", [(2, (2, 0, 2)), (2, (1, 0, 0, 1, 0, 3)), (2, (0, 3, 1, 0, 1)),
                                          (3, (2, 0, 2)), (3, (1, 0, 1, 1)), (2, (4,))])
@pytest.mark.parametrize("first", [1, 2])
def test_no_order_of_steps_loses_a_word(model, members, jobs, first):
    res = model(members, False, first, jobs)
    assert res.returncode == 0 and res.stdout.startswith("states"), res.stdout


def test_a_number_for_a_subdomain_without_a_sweep_loses_one(model):
    """What the rule rules out: the first sweep after a skipped subdomain would
    overwrite the last one before it, which a neighbour may still wait for."""
    res = model(2, True, 1, (2, 0, 2))
    assert res.returncode == 1 and "stuck" in res.stdout


@pytest.mark.parametrize("jobs,teams", [(1, 1), (512, 64), (512, 512), (32768, 1), (7, 9)])
@pytest.mark.parametrize("max_inner", [1, 500, 4000, 1 << 20, (1 << 29) - 1, 1 << 29, (1 << 31) - 1])
def test_no_number_is_used_twice_between_clears(model, jobs, teams, max_inner):
    """Each launch between two clears of the mailboxes has numbers of its own,
    for every sweep that a team can make (up to 2^31 of them), and none is 0, which
    cleared words hold."""
    span, launches, first = model.numbers(jobs, teams, max_inner, 1)
    most = (max(0, jobs - teams) + 1) * (max_inner + 1)
    assert span == min(most, 1 << 31)
    assert launches >= 1 and first == 1
    for launch in {1, 2, min(launches, 4096), launches}:
        if launch <= launches:
            lo = model.numbers(jobs, teams, max_inner, launch)[2]
            assert lo == 1 + (launch - 1) * span and lo + span - 1 < 1 << 32
