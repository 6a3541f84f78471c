"""Entries of the tuning cache (needs an MI355X): contexts whose options, condition
or rows allow other kernels do not read or replace each other's."""
import json

import pytest

from bridge import Case, gpu_available
from test_gpu_chip import _forced

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

OPTS = dict(precision="fp32", mode="batched", inner_tol=1e-2, inner_abs=0.0, check_every=10, max_outer=20000)


@pytest.mark.parametrize("other", [dict(resident=0), dict(q=0.004)])
def test_another_kind_of_context_keeps_its_own_entry(other, tmp_path, monkeypatch):
    case = Case(ne=(32, 32, 32), cuts=((16,), (16,), (16,)), p=16.0)
    prob, d = _forced(case, 4, tmp_path, monkeypatch, **OPTS)
    prob.solve(d, 1e-8)
    prob.close()
    cache = tmp_path / "tune.jsonl"
    prob = case.problem(**OPTS, **other)
    _, st = prob.solve(d, 1e-8)
    prob.close()
    assert "resident" not in other or st["resident"] != 3
    keys = [json.loads(v)["key"] for v in cache.read_text().splitlines()]
    assert len(keys) == 2 and keys[0] != keys[1]
    prob = case.problem(**OPTS)
    _, st = prob.solve(d, 1e-8)
    prob.close()
    assert st["resident"] == 3 and st["team"] == 4
    assert len(cache.read_text().splitlines()) == 2


def test_rows_that_start_elsewhere_are_another_geometry(tmp_path, monkeypatch):
    """The same node counts, a Neumann face at the low or at the high end of x."""
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("SOS_TUNE_CACHE", str(cache))
    import torch
    for bc in ((1, 0, 0, 0, 0, 0), (0, 1, 0, 0, 0, 0)):
        case = Case(ne=(5, 6, 6), bc=bc, cuts=((), (3,), ()), p=11.0)
        prob = case.problem(**OPTS)
        prob.solve(torch.ones(5 * 6 * 6, dtype=torch.float64, device="cuda"), 1e-6)
        prob.close()
    keys = [json.loads(v)["key"] for v in cache.read_text().splitlines()]
    assert len(keys) == 2 and keys[0] != keys[1]


def test_streaming_shape_stays_known_beside_the_on_chip_form(tmp_path, monkeypatch):
    """Unequal teams set on a context that the tuner gave the on-chip form run with
    the tuner's streaming shape, found or read from the cache, as on a context that it
    gave the streaming form."""
    import numpy as np
    import torch
    from synth.generators import uniform_density
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("SOS_TUNE_CACHE", str(cache))
    case = Case(ne=(48, 48, 48), cuts=((16, 32), (16, 32), (16, 32)), p=16.0)
    opts = dict(OPTS, precision="fp64", inner_tol=1e-3)
    d = torch.tensor(uniform_density(case.ne, seed=3), device="cuda")
    teams = np.where(np.arange(case.part.n_sub) % 2, 1, 2)
    for k in range(2):  # the search, then its cached entry
        prob = case.problem(**opts)
        _, st = prob.solve(d, 1e-6)
        assert st["resident"] == 3  # (390 against 880 ms a solve)
        entry = json.loads(cache.read_text())
        threads, cpt, rows, resident = entry["streaming"]
        prob.set_teams(teams)
        _, st = prob.solve(d, 1e-6)
        assert (st["block"], st["cols_per_thread"], st["wave_rows"], st["team"]) == (threads, cpt, rows, 2), (k, entry)
        assert st["resident"] != 3 and st["converged"]
        prob.close()
