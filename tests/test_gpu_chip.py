"""The fused CG kernel with the whole state of an inner solve on the chip (needs
an MI355X): every kernel variant (planes per block, teams, first and last node
of a row a vertex or a mid-point, idle lanes and rows, second-order terms, FP32
and FP64) against the oracle. The variant is forced through the tuning cache."""
import json

import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from oracle import direct as D
from oracle import schwarz as S
from synth.generators import uniform_density

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _forced(case, team, tmp_path, monkeypatch, **kw):
    """A problem whose first solve takes the on-chip form with this team size:
    the tuning cache entry of the same geometry, rewritten."""
    import torch
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("SOS_TUNE_CACHE", str(cache))
    d = torch.tensor(uniform_density(case.ne, seed=3), device="cuda")
    first = case.problem(**dict(kw, max_outer=1))
    first.solve(d, 1e-30)
    first.close()
    line = json.loads(cache.read_text().splitlines()[-1])
    line.update(threads=0, cpt=2, teams=[team] * len(line["teams"]), rows=1, resident=3)
    cache.write_text(json.dumps(line) + "\n")
    return case.problem(**kw), d


# x and y node counts with either end a vertex or a mid-point, one-node-thick
# axes, teams down to two planes a member
STEP = {
    "ragged_team1": (dict(ne=(6, 5, 6), bc=(0, 0, 1, 0, 0, 0), cuts=((3,), (2,), (2, 4)), p=11.0), 1),
    "ragged_team2": (dict(ne=(7, 6, 5), lengths=(1.0, 0.8, 1.3), bc=(0, 1, 0, 0, 1, 0),
                          cuts=((2, 3), (4,), (2,)), p=5.5), 2),
    "columns_team8": (dict(ne=(5, 4, 9), bc=(1, 0, 0, 1, 0, 0), cuts=((2,), (2,), ()), p=24.0), 8),
    "one_node_rows": (dict(ne=(1, 6, 5), cuts=((), (3,), ()), p=30.0), 3),
    "one_row": (dict(ne=(6, 1, 5), cuts=((2,), (), ()), p=30.0), 2),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("q", [0.0, 0.02])
@pytest.mark.parametrize("name", sorted(STEP))
def test_one_outer_iteration_on_chip_matches_oracle(name, q, prec, tmp_path, monkeypatch):
    """u^1 and lambda^1 from a random state against the oracle's LU solves:
    FP64 to 1e-10, FP32 inner solves (to 1e-6 of r) to 1e-4."""
    import torch
    kw, team = STEP[name]
    case = Case(**kw)
    opts = dict(inner_tol=1e-30, inner_abs=1e-14) if prec == "fp64" else dict(inner_tol=1e-6, inner_abs=0.0)
    prob, d = _forced(case, team, tmp_path, monkeypatch, precision=prec, mode="batched", q=q, max_inner=4000,
                      max_outer=1, **opts)
    _, st = prob.solve(d, 1e-30)
    print("case", name, prec, "q", q, "block", st["block"], "team", st["team"], flush=True)
    assert st["resident"] == 3 and st["team"] == team
    lay = case.check_layout(prob)
    f, fs = case.density_loads(d.cpu().numpy())
    rng = np.random.default_rng(5)
    u0 = [1e-9 * rng.standard_normal(s.n) for s in case.part.subs]
    lam0 = [1e-10 * rng.standard_normal(fc.nodes.size) for fc in case.part.faces]
    prob.set_state(torch.tensor(case.to_local(lay, u0), device="cuda"),
                   torch.tensor(case.faces_to_lam(lay, lam0), device="cuda"))
    prob.iterate(1)
    u1, lam1 = prob.get_state()
    u1 = case.from_local(lay, u1.cpu().numpy())
    lam1 = case.lam_to_faces(lay, lam1.cpu().numpy())
    prob.close()
    orc = S.SchwarzOracle(case.part, case.p, "lu", q_face=q)
    ur = orc.subdomain_solves(fs, lam0)
    lr = orc.exchange(ur, lam0)
    bound = 1e-10 if prec == "fp64" else 1e-4
    for s in range(case.part.n_sub):
        assert np.abs(u1[s] - ur[s]).max() <= bound * np.abs(ur[s]).max(), s
    for fc in range(len(lr)):
        assert np.abs(lam1[fc] - lr[fc]).max() <= bound * np.abs(lr[fc]).max(), fc


# 32 or 33 nodes a row (17 pairs, the kernels compiled for that) and others, at the most planes of each variant; more teams than fit at once
SOLVES = {
    "plane33_17_planes": (dict(ne=(32, 32, 34), cuts=((16,), (16,), (17,)), p=16.0), "fp32", 2),
    "plane33_11_planes": (dict(ne=(48, 48, 48), cuts=((16, 32), (16, 32), (16, 32)), p=16.0), "fp32", 3),
    "plane30_12_planes": (dict(ne=(30, 30, 36), cuts=((15,), (15,), (18,)), p=16.0), "fp32", 3),
    "plane33_9_planes": (dict(ne=(48, 48, 18), cuts=((16, 32), (16, 32), ()), p=16.0), "fp32", 4),
    "plane33_5_planes": (dict(ne=(48, 48, 20), cuts=((16, 32), (16, 32), ()), p=16.0), "fp32", 8),
    "plane33_fp64": (dict(ne=(48, 48, 20), cuts=((16, 32), (16, 32), ()), p=16.0), "fp64", 8),
    "plane21_17_planes": (dict(ne=(20, 20, 17), cuts=((10,), (10,), ()), p=16.0), "fp32", 2),
    "team16_3_planes": (dict(ne=(32, 32, 24), cuts=((16,), (16,), ()), p=16.0), "fp32", 16),
    "team48_slab": (dict(ne=(20, 18, 52), lengths=(1.0, 1.0, 3.0), cuts=((5, 10, 15), (), ()), p=20.0), "fp32", 48),
    "team24_fp64": (dict(ne=(20, 18, 52), lengths=(1.0, 1.0, 3.0), cuts=((5, 10, 15), (), ()), p=20.0), "fp64", 24),
    "many_teams": (dict(ne=(60, 60, 12), cuts=(tuple(range(5, 60, 5)), tuple(range(5, 60, 5)), (3, 6, 9)), p=24.0),
                   "fp32", 3),
}


@pytest.mark.parametrize("q", [0.0, 0.004])
@pytest.mark.parametrize("name", sorted(SOLVES))
def test_solve_on_chip_matches_direct(name, q, tmp_path, monkeypatch):
    """Whole solves to 1e-10: the oracle's residual meets the tolerance, the
    solution is the direct one to 20 tol (the bound of the largest-plane solves)
    and graph replays and eager launches agree bit for bit."""
    import torch
    kw, prec, team = SOLVES[name]
    case = Case(**kw)
    opts = dict(precision=prec, mode="batched", q=q, inner_tol=1e-2, inner_abs=0.0, check_every=10, max_outer=20000)
    prob, d = _forced(case, team, tmp_path, monkeypatch, **opts)
    phi, st = prob.solve(d, 1e-10)
    prob.set_opts(use_graph=0)
    phi2, st2 = prob.solve(d, 1e-10)
    prob.close()
    print("case", name, "q", q, "outer", st["outer_iters"], "inner", st["inner_iters"], "block", st["block"], flush=True)
    assert st["resident"] == 3 and st["team"] == team and st["converged"]
    assert torch.equal(phi, phi2) and st["inner_iters"] == st2["inner_iters"]
    f, _ = case.density_loads(d.cpu().numpy())
    ud = D.solve_direct(case.mesh, f, "fdm")
    phi = phi.cpu().numpy()
    err = np.abs(phi - ud).max() / np.abs(ud).max()
    res = A.residual_norm(case.mesh, phi, f)
    print("residual", res, "err", err, flush=True)
    assert res <= 1e-10 * 1.001 and err <= 20 * 1e-10


def test_unequal_teams_leave_the_chip_form(tmp_path, monkeypatch):
    """One team size for all subdomains: other teams set by the caller are taken
    by the form that has them."""
    import torch
    case = Case(ne=(24, 20, 16), cuts=((3, 8, 15), (4, 11), ()), p=160.0)
    prob, d = _forced(case, 2, tmp_path, monkeypatch, precision="fp32", mode="batched", check_every=5,
                      max_outer=20000, inner_tol=1e-2, inner_abs=0.0)
    _, st = prob.solve(d, 1e-8)
    assert st["resident"] == 3 and st["team"] == 2
    teams = np.where(np.arange(case.part.n_sub) % 2, 1, 2)
    prob.set_teams(teams)
    phi, st = prob.solve(d, 1e-8)
    assert st["resident"] != 3 and np.array_equal(prob.teams(), teams) and st["converged"]
    f, _ = case.density_loads(d.cpu().numpy())
    assert A.residual_norm(case.mesh, phi.cpu().numpy(), f) <= 1e-8 * 1.001
    prob.set_robin(160.0, 0.001)
    phi, st = prob.solve(d, 1e-8)
    assert st["converged"]
    prob.close()


def test_teams_of_another_context(tmp_path, monkeypatch):
    """Teams of more than eight members, as one context reports them, are taken
    by a fresh one; unequal ones of that size are refused."""
    import torch
    from paper_2112_03851_amd.sos import SosError
    kw, prec, team = SOLVES["team48_slab"]
    case = Case(**kw)
    opts = dict(precision=prec, mode="batched", check_every=10, max_outer=20000, inner_tol=1e-2, inner_abs=0.0)
    prob, d = _forced(case, team, tmp_path, monkeypatch, **opts)
    phi, st = prob.solve(d, 1e-8)
    teams = prob.teams()
    prob.close()
    other = case.problem(**opts)
    bad = np.array(teams)
    bad[0] = 9
    with pytest.raises(SosError):
        other.set_teams(bad)
    other.set_teams(teams)
    phi2, st2 = other.solve(d, 1e-8)
    assert st["team"] == st2["team"] == team and st2["resident"] == 3 and torch.equal(phi, phi2)
    other.close()
