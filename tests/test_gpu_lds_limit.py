"""LDS at its limit (needs an MI355X): a workgroup's static LDS counts towards
the 160 KB, so a resident vector that fits beside the march planes alone stays
out of LDS."""
import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from synth.generators import uniform_density

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def test_resident_x_leaves_room_for_static_lds():
    """32x32x36-node subdomains: x and three march planes take 163,008 of
    163,840 bytes, the kernel's own sums 1,120: x does not stay in LDS. One plane
    less (z cut one element lower on the other side) it does."""
    import torch
    for ne, cut, level in (((32, 32, 36), 18, 0), ((32, 32, 35), 18, 0), ((32, 32, 34), 17, 2)):
        case = Case(ne=ne, cuts=((16,), (16,), (cut,)), p=16.0)
        drho = uniform_density(case.ne, seed=2)
        prob = case.problem(precision="fp32", mode="batched", block=1024, team=1, resident=1, check_every=10,
                            inner_tol=1e-2, inner_abs=0.0, max_outer=20000)
        phi, st = prob.solve(torch.tensor(drho, device="cuda"), 1e-8)
        prob.close()
        print(ne, "planes", max(s.shape[2] for s in case.part.subs), "resident", st["resident"], flush=True)
        assert st["resident"] == level and st["converged"]
        f, _ = case.density_loads(drho)
        assert A.residual_norm(case.mesh, phi.cpu().numpy(), f) <= 1e-8 * 1.001
        assert np.isfinite(phi.cpu().numpy()).all()
