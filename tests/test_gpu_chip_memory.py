"""No memory for the workspace of the on-chip fused CG (needs an MI355X): runs take
the streaming form, which needs none, and the context stays whole."""
import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from paper_2112_03851_amd import sos
from synth.generators import uniform_density
from test_gpu_chip import SOLVES, _forced

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

OPTS = dict(precision="fp32", mode="batched", inner_tol=1e-2, inner_abs=0.0, check_every=10, max_outer=20000)
PLANES32 = dict(ne=(32, 32, 32), cuts=((16,), (16,), (16,)), p=16.0)


def _solves(case, prob, d, resident):
    phi, st = prob.solve(d, 1e-9)
    f, _ = case.density_loads(d.cpu().numpy())
    assert st["converged"] and (st["resident"] == 3) == resident, st
    assert A.residual_norm(case.mesh, phi.cpu().numpy(), f) <= 1e-9 * 1.001
    return phi, st


def test_tuner_drops_the_candidate(tmp_path, monkeypatch):
    """The search goes on without the on-chip form, and what it finds then is not
    kept for contexts that have the memory."""
    import torch
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("SOS_TUNE_CACHE", str(cache))
    case = Case(**PLANES32)
    d = torch.tensor(uniform_density(case.ne, seed=3), device="cuda")
    prob = case.problem(**OPTS)
    prob.debug_workspace(1)
    _solves(case, prob, d, False)
    _solves(case, prob, d, False)
    assert not cache.exists()
    prob.close()


def test_cached_form_without_memory(tmp_path, monkeypatch):
    case = Case(**PLANES32)
    prob, d = _forced(case, 4, tmp_path, monkeypatch, **OPTS)
    before = (tmp_path / "tune.jsonl").read_text()
    prob.debug_workspace(1)
    _solves(case, prob, d, False)
    assert (tmp_path / "tune.jsonl").read_text() == before
    prob.close()
    again = case.problem(**OPTS)
    _solves(case, again, d, True)
    again.close()


def test_memory_that_runs_out_on_a_used_context(tmp_path, monkeypatch):
    """A replan (another condition) or more teams that need a workspace there is no
    memory for: solves, iterations and new teams go on in the streaming form."""
    import torch
    case = Case(**PLANES32)
    prob, d = _forced(case, 4, tmp_path, monkeypatch, **OPTS)
    phi, _ = _solves(case, prob, d, True)
    prob.debug_workspace(1)
    prob.set_robin(case.p, 0.004)
    _solves(case, prob, d, False)
    prob.set_robin(case.p, 0.0)
    _solves(case, prob, d, False)
    prob.close()

    prob = case.problem(**OPTS)
    phi2, _ = _solves(case, prob, d, True)
    assert torch.equal(phi, phi2)
    prob.debug_workspace(1)
    st = prob.iterate(3)
    assert st["resident"] != 3 and np.isfinite(st["rel_residual"])
    prob.close()

    prob = case.problem(**OPTS)
    _solves(case, prob, d, True)
    prob.debug_workspace(1)
    prob.set_teams(np.full(case.part.n_sub, 2))
    _, st = _solves(case, prob, d, False)
    assert st["team"] == 2
    prob.debug_workspace(0)
    prob.close()


def test_large_teams_without_memory(tmp_path, monkeypatch):
    """Teams of more than eight exist on the chip alone: SOS_ENOMEM, and the
    context solves as before."""
    kw, prec, team = SOLVES["team48_slab"]
    case = Case(**kw)
    prob, d = _forced(case, team, tmp_path, monkeypatch, **OPTS)
    _solves(case, prob, d, True)
    teams = prob.teams()
    prob.close()
    prob = case.problem(**dict(OPTS, resident=1))
    prob.debug_workspace(1)
    with pytest.raises(sos.SosError) as ei:
        prob.set_teams(teams)
    assert ei.value.code == sos.SOS_ENOMEM
    _solves(case, prob, d, False)
    prob.debug_workspace(0)
    prob.set_teams(teams)
    _, st = _solves(case, prob, d, True)
    assert st["team"] == team
    prob.close()


def test_options_refused_leave_the_context_whole(tmp_path, monkeypatch):
    """A block that cannot cover the plane is refused; the context solves on."""
    case = Case(**PLANES32)
    prob, d = _forced(case, 4, tmp_path, monkeypatch, **OPTS)
    _solves(case, prob, d, True)
    with pytest.raises(sos.SosError):
        prob.set_opts(block=64, resident=0)
    _solves(case, prob, d, False)
    prob.set_opts(block=0, resident=1)
    _solves(case, prob, d, True)
    prob.close()
