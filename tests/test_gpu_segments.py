"""z-segments of the residual, check and plain CG kernels on a small problem
(needs an MI355X): segments of two and four planes, a remainder of one, and
more than 64 blocks in a subdomain, against the direct solution."""
import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from oracle import direct as D
from synth.generators import uniform_density

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

CASES = {
    "two_planes_71_blocks": dict(ne=(4, 5, 72), lengths=(1.0, 1.2, 9.0), cuts=((2,), (), ()), p=8.0),
    "four_planes_remainder": dict(ne=(40, 6, 11), cuts=(tuple(range(1, 40)), (), ()), p=40.0),
    "one_plane": dict(ne=(6, 7, 1), cuts=((3,), (2,), ()), p=24.0),
}


@pytest.mark.parametrize("form,prec,q", [("stepwise", "fp64", 0.0), ("stepwise", "fp32", 0.01), ("batched", "fp32", 0.01)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_short_segments_match_direct(name, form, prec, q):
    """Whole solves to 1e-9: the oracle's residual meets the tolerance, the
    solution is the direct one to 20 tol (the bound of the other whole solves)."""
    import torch
    case = Case(**CASES[name])
    d = torch.tensor(uniform_density(case.ne, seed=3), device="cuda")
    prob = case.problem(precision=prec, mode=form, q=q, inner_tol=1e-2, inner_abs=0.0, check_every=10, max_outer=20000)
    phi, st = prob.solve(d, 1e-9)
    prob.close()
    print("case", name, form, prec, "outer", st["outer_iters"], flush=True)
    f, _ = case.density_loads(d.cpu().numpy())
    ud = D.solve_direct(case.mesh, f, "fdm")
    phi = phi.cpu().numpy()
    res = A.residual_norm(case.mesh, phi, f)
    err = np.abs(phi - ud).max() / np.abs(ud).max()
    print("residual", res, "err", err, flush=True)
    assert st["converged"] and res <= 1e-9 * 1.001 and err <= 20 * 1e-9
