"""Waits of the on-chip fused CG that end at their bound (needs an MI355X): the sums'
and the mailboxes' time-outs, the members' return, and the context afterwards."""
import pytest

from bridge import Case, gpu_available
from paper_2112_03851_amd import sos
from test_gpu_chip import _forced
from test_gpu_chip_jobs import JOBS

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

CASES = {
    "one_job_each": (dict(ne=(16, 16, 16), cuts=((8,), (8,), ()), p=128.0), "fp32", 4),
    "fp64": (dict(ne=(16, 16, 16), cuts=((8,), (8,), ()), p=128.0), "fp64", 8),
    "jobs_in_turn": (JOBS["equal"], "fp32", 3),
}


@pytest.mark.parametrize("graph", [1, 0])
@pytest.mark.parametrize("name", sorted(CASES))
def test_waits_that_never_succeed_report_breakdown(name, graph, tmp_path, monkeypatch):
    """Every member waits for a tag and for mail that nobody writes, at most 20,000
    ticks (0.2 ms; 64 times that for the first meeting of a launch): the solve stops with
    SOS_EBREAKDOWN at its first check, and the context then solves as a fresh one
    does, bit for bit."""
    import torch
    kw, prec, team = CASES[name]
    case = Case(**kw)
    opts = dict(precision=prec, mode="batched", inner_tol=1e-2, inner_abs=0.0, check_every=4, max_outer=20000,
                use_graph=graph)
    prob, d = _forced(case, team, tmp_path, monkeypatch, **opts)
    fresh, st = prob.solve(d, 1e-8)
    assert st["resident"] == 3 and st["team"] == team
    prob.debug_barrier(spin_ticks=20000, tag_skew=1)
    print("case", name, "graph", graph, "waits forced to give up", flush=True)
    with pytest.raises(sos.SosError) as ei:
        prob.solve(d, 1e-8)
    assert ei.value.code == sos.SOS_EBREAKDOWN and "team barrier" in str(ei.value)
    hist = prob.history()
    assert len(hist) == 1 and hist[0][0] == 4
    prob.debug_barrier(0, 0)
    phi, st2 = prob.solve(d, 1e-8)
    prob.close()
    assert st2["resident"] == 3 and st2["inner_iters"] == st["inner_iters"] and torch.equal(phi, fresh)
