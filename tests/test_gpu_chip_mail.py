"""The on-chip fused CG on a context that has been used before (needs an MI355X):
mailboxes that lie where another team size kept its vectors, sequence numbers that
run out, and transmission conditions that change the kernel."""
import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from oracle import direct as D
from test_gpu_chip import _forced

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# 32 planes of 32 x 32 nodes: teams of two keep w and x in the workspace too
PLANES32 = dict(ne=(32, 32, 32), cuts=((16,), (16,), (16,)), p=16.0)
OPTS = dict(precision="fp32", mode="batched", inner_tol=1e-2, inner_abs=0.0, check_every=10, max_outer=20000)


def _check(case, d, phi, tol):
    f, _ = case.density_loads(d.cpu().numpy())
    ud = D.solve_direct(case.mesh, f, "fdm")
    phi = phi.cpu().numpy()
    assert A.residual_norm(case.mesh, phi, f) <= tol * 1.001
    assert np.abs(phi - ud).max() <= 20 * tol * np.abs(ud).max()


def test_team_sizes_changed_on_one_context(tmp_path, monkeypatch):
    """Each solve equals that of a fresh context with the same teams, bit for bit."""
    import torch
    case = Case(**PLANES32)
    used, d = _forced(case, 4, tmp_path, monkeypatch, **OPTS)
    used.solve(d, 1e-10)
    for team in (4, 2, 3, 2, 6, 4):
        used.set_teams(np.full(case.part.n_sub, team))
        phi, st = used.solve(d, 1e-10)
        (tmp_path / "tune.jsonl").unlink(missing_ok=True)
        fresh, _ = _forced(case, team, tmp_path, monkeypatch, **OPTS)
        phi2, st2 = fresh.solve(d, 1e-10)
        fresh.close()
        print("team", team, "outer", st["outer_iters"], flush=True)
        assert st["team"] == st2["team"] == team and st["resident"] == st2["resident"] == 3
        assert st["inner_iters"] == st2["inner_iters"] and torch.equal(phi, phi2)
    used.close()
    _check(case, d, phi, 1e-10)


@pytest.mark.parametrize("team", [2, 3])
def test_sequence_numbers_run_out(team, tmp_path, monkeypatch):
    """An iteration limit so large that the mailboxes are cleared before every
    launch, or within each graph of ten: the same solve as with the usual limit, in
    graphs and in eager launches."""
    import torch
    case = Case(**PLANES32)
    want = None
    for max_inner in (500, 2**31 - 1, 2**29):
        (tmp_path / "tune.jsonl").unlink(missing_ok=True)
        prob, d = _forced(case, team, tmp_path, monkeypatch, max_inner=max_inner, **OPTS)
        for graph in (1, 0):
            prob.set_opts(use_graph=graph)
            phi, st = prob.solve(d, 1e-10)
            assert st["resident"] == 3 and st["team"] == team and st["converged"]
            got = (st["outer_iters"], st["inner_iters"])
            if want is None:
                want = got, phi
            assert got == want[0] and torch.equal(phi, want[1]), (max_inner, graph)
        prob.close()
    _check(case, d, want[1], 1e-10)


def test_iteration_limit_changed_on_one_context(tmp_path, monkeypatch):
    """Another limit sets aside another span of numbers for each launch."""
    import torch
    case = Case(**PLANES32)
    prob, d = _forced(case, 3, tmp_path, monkeypatch, **OPTS)
    phi, _ = prob.solve(d, 1e-10)
    for max_inner in (70, 2**29, 500):
        prob.set_opts(max_inner=max_inner)
        phi2, st = prob.solve(d, 1e-10)
        assert st["resident"] == 3 and torch.equal(phi, phi2), max_inner
    prob.close()


def test_order_of_the_condition_changed_on_one_context(tmp_path, monkeypatch):
    """Zeroth to second order and back: another kernel variant, replanned."""
    import torch
    case = Case(**PLANES32)
    used, d = _forced(case, 3, tmp_path, monkeypatch, **OPTS)
    zeroth, st = used.solve(d, 1e-10)
    used.set_robin(case.p, 0.004)
    second, st2 = used.solve(d, 1e-10)
    used.set_robin(case.p, 0.0)
    back, st3 = used.solve(d, 1e-10)
    used.close()
    assert st["resident"] == st2["resident"] == st3["resident"] == 3
    assert torch.equal(zeroth, back) and st["inner_iters"] == st3["inner_iters"]
    (tmp_path / "tune.jsonl").unlink()
    fresh, _ = _forced(case, 3, tmp_path, monkeypatch, q=0.004, **OPTS)
    want, _ = fresh.solve(d, 1e-10)
    fresh.close()
    assert torch.equal(second, want)
    _check(case, d, second, 1e-10)
