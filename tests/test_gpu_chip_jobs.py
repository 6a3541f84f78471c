"""Persistent teams of the on-chip fused CG that take several subdomains in turn
(needs an MI355X): subdomains that need no sweep between others, subdomains of
different shape."""
import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from oracle import direct as D
from test_gpu_chip import _forced

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _cuts(widths):
    return tuple(int(v) for v in np.cumsum(widths)[:-1])


# more subdomains than teams that the GPU holds at once (three blocks a compute
# unit at most, so 256 teams of three)
FIVES = _cuts([5] * 12)
MIXED = [2, 5, 3, 4] * 5
JOBS = {
    "equal": dict(ne=(60, 60, 12), cuts=(FIVES, FIVES, (3, 6, 9)), p=24.0),
    "uneven": dict(ne=(sum(MIXED), sum(MIXED), 8), lengths=(1.0, 1.0, 0.3), cuts=(_cuts(MIXED), _cuts(MIXED[::-1]), ()),
                   p=60.0),
}


@pytest.mark.parametrize("prec,abs_tol", [("fp32", 0.0), ("fp32", 1e-11), ("fp64", 0.0)])
@pytest.mark.parametrize("name", sorted(JOBS))
def test_subdomains_that_need_no_sweep(name, prec, abs_tol, tmp_path, monkeypatch):
    """A density of a few elements in one corner: in the first outer iterations
    most residuals are exactly zero, and with an absolute tolerance more and more
    already meet it, so teams skip subdomains between others. Against the direct
    solution (20 tol, as the other whole solves), and bit for bit in the fixed and
    in the work order of the subdomains, which pair other skips."""
    import torch
    case = Case(**JOBS[name])
    opts = dict(precision=prec, mode="batched", inner_tol=1e-2, inner_abs=abs_tol, check_every=5, max_outer=20000)
    prob, _ = _forced(case, 3, tmp_path, monkeypatch, **opts)
    rho = np.zeros(case.ne[::-1])
    rho[:2, :3, :2] = 250.0
    rho[-1, 1, 1] = -90.0
    d = torch.tensor(rho.ravel(), device="cuda")
    print("case", name, prec, abs_tol, flush=True)
    phi, st = prob.solve(d, 1e-9)
    prob.set_opts(schedule=0)
    phi2, st2 = prob.solve(d, 1e-9)
    prob.close()
    print("outer", st["outer_iters"], "inner", st["inner_iters"], flush=True)
    assert st["resident"] == 3 and st["team"] == 3 and st["converged"]
    assert st["inner_iters"] == st2["inner_iters"] and torch.equal(phi, phi2)
    f, _ = case.density_loads(rho.ravel())
    ud = D.solve_direct(case.mesh, f, "fdm")
    phi = phi.cpu().numpy()
    assert A.residual_norm(case.mesh, phi, f) <= 1e-9 * 1.001
    assert np.abs(phi - ud).max() <= 20 * 1e-9 * np.abs(ud).max()


def test_a_subdomain_without_a_sweep_is_left_alone(tmp_path, monkeypatch):
    """One outer iteration from zero: subdomains without a source keep u = 0 and
    count no iteration."""
    import torch
    case = Case(**JOBS["equal"])
    prob, _ = _forced(case, 3, tmp_path, monkeypatch, precision="fp32", mode="batched", inner_tol=1e-2,
                      max_outer=1)
    rho = np.zeros(case.ne[::-1])
    rho[:2, :3, :2] = 250.0
    prob.solve(torch.tensor(rho.ravel(), device="cuda"), 1e-30)
    iters = prob.inner_iters()
    u, _ = prob.get_state()
    lay = prob.layout()
    prob.close()
    u = u.cpu().numpy()
    zero = [not u[lay["offsets"][s]:lay["offsets"][s] + int(np.prod(lay["dims"][s]))].any()
            for s in range(case.part.n_sub)]
    assert iters[0] > 0 and not zero[0]
    assert all(zero[1:]) and not np.any(np.asarray(iters)[1:])
