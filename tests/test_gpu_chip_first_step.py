"""The first step length of an FP32 inner solve in the on-chip fused CG (needs an
MI355X): gamma = r'D^-1 r and delta = w'D^-1 r of the start are FP64 products and
sums, as in the streaming form."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla
from scipy.sparse import diags

from bridge import Case, gpu_available
from oracle import subdomain as SD
from test_gpu_chip import _forced

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("team,planes", [(2, 17), (3, 12)])
def test_first_step_of_an_fp32_solve(team, planes, tmp_path, monkeypatch):
    """A residual of random signs with r_i^2 / D_ii = 1 + 0.8 2^-20 at every node:
    summed in FP32 over a thread's 2 x 17 (12) nodes, each addition past 16 drops
    the excess, 2.5e-7 to 3.6e-7 of gamma and so of the step. From the step that u
    took, against FP64 sums: its own rounding to FP32 (2^-24), and 5e-8 for the FP32
    rounding of w, which random signs average out over 30,000 nodes."""
    import torch
    case = Case(ne=(15, 15, 34 if team == 2 else 36), cuts=((), (), (17,) if team == 2 else (18,)), p=16.0)
    prob, _ = _forced(case, team, tmp_path, monkeypatch, precision="fp32", mode="batched", inner_tol=1e-30, max_inner=1,
                      max_outer=1)
    rho = np.ones(int(np.prod(case.ne)))
    _, st = prob.solve(torch.tensor(rho, device="cuda"), 1e-30)
    assert st["resident"] == 3 and st["team"] == team
    _, fs = case.density_loads(rho)
    lay = case.check_layout(prob)
    rng = np.random.default_rng(11)
    mats = [SD.robin_matrix(case.part, sub, lambda f: case.p) for sub in case.part.subs]
    r, u0 = [], []
    for M, f in zip(mats, fs):
        v = np.sqrt(M.diagonal() * (1.0 + 0.8 * 2.0**-20)) * np.where(rng.random(M.shape[0]) < 0.5, -1.0, 1.0)
        r.append(v.astype(np.float32).astype(float))
        u, info = spla.cg(M, f - r[-1], rtol=1e-12, maxiter=5000, M=diags(1.0 / M.diagonal()))
        assert info == 0
        u0.append(u)
    lam = torch.zeros(max(1, int(lay["face_off"][-1])), dtype=torch.float64, device="cuda")
    prob.set_state(torch.tensor(case.to_local(lay, u0), device="cuda"), lam)
    prob.iterate(1)
    u1 = case.from_local(lay, prob.get_state()[0].cpu().numpy())
    prob.close()
    for s, M in enumerate(mats):
        u = r[s] / M.diagonal()
        want = (r[s] @ u) / (u @ (M @ u))
        step = u1[s] - u0[s]
        got = (step @ r[s]) / (u @ r[s])  # (weights in which the rounding of 1 / D_ii cancels)
        print("subdomain", s, "planes", planes, "step", got, "off by", got / want - 1.0, flush=True)
        assert np.abs(step - got * u).max() <= 1e-6 * np.abs(got * u).max()  # (it is a multiple of D^-1 r)
        assert abs(got / want - 1.0) <= 2.0**-24 + 5e-8
