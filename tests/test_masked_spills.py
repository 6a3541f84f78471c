"""Register spills under a partial lane mask: the build finds them in a kernel's
assembly, and the FP64 kernel that had one (four columns a thread, two segments
a block, second-order terms, teams) solves what it broke down on."""
import json

import numpy as np
import pytest

from bridge import Case, gpu_available
from oracle import assemble as A
from oracle import direct as D
from paper_2112_03851_amd.build import masked_spills
from synth.generators import uniform_density

LOOP = """
_Z3foo:
; %%bb.0:
\ts_and_saveexec_b64 s[2:3], vcc
\ts_cbranch_execz .LBB0_3
; %%bb.1:
\tds_write_b64 v4, v[2:3]
\ts_andn2_b64 exec, exec, s[10:11]
\ts_cbranch_execnz .LBB0_2
.LBB0_3:                              ; %%exit
\tv_writelane_b32 v167, s67, 43
%s\ts_or_b64 exec, exec, s[2:3]
%s\ts_endpgm
"""
SPILL = "\tscratch_store_dword off, v38, off offset:24 ; 4-byte Folded Spill\n"


def test_spill_before_the_mask_is_restored_is_found():
    assert masked_spills(LOOP % (SPILL, "")) == [("_Z3foo", "scratch_store_dword off, v38, off offset:24")]
    assert masked_spills(LOOP % ("\tv_mov_b32_e32 v1, v2\n", "")) == [("_Z3foo", "v_mov_b32_e32 v1, v2")]
    assert masked_spills(LOOP % ("", SPILL)) == []
    exit_only = (LOOP % (SPILL, "")).replace(".LBB0_3:", "; %bb.3:")
    assert masked_spills(exit_only) == [("_Z3foo", "scratch_store_dword off, v38, off offset:24")]


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("team", [2, 4])
def test_fp64_four_columns_two_segments(team, tmp_path, monkeypatch):
    """The whole solve against the direct solution (20 tol, as for the other
    whole solves); the shape is forced through the tuning cache."""
    import torch
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("SOS_TUNE_CACHE", str(cache))
    case = Case(ne=(48, 48, 48), cuts=((16, 32), (16, 32), (16, 32)), p=16.0)
    opts = dict(precision="fp64", mode="batched", q=0.01, inner_tol=1e-3, inner_abs=0.0, check_every=10)
    d = torch.tensor(uniform_density(case.ne, seed=3), device="cuda")
    first = case.problem(**opts, max_outer=1)
    first.solve(d, 1e-30)
    first.close()
    line = json.loads(cache.read_text().splitlines()[-1])
    line.update(threads=640, cpt=4, teams=[team] * len(line["teams"]), rows=0, resident=0)
    cache.write_text(json.dumps(line) + "\n")
    prob = case.problem(**opts, max_outer=20000)
    phi, st = prob.solve(d, 1e-10)
    prob.close()
    assert st["block"] == 640 and st["cols_per_thread"] == 4 and st["team"] == team and st["converged"]
    f, _ = case.density_loads(d.cpu().numpy())
    ud = D.solve_direct(case.mesh, f, "fdm")
    phi = phi.cpu().numpy()
    assert A.residual_norm(case.mesh, phi, f) <= 1e-10 * 1.001
    assert np.abs(phi - ud).max() <= 20 * 1e-10 * np.abs(ud).max()
