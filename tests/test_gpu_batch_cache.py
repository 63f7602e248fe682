"""A schedule index that another version stored in BSI_TUNE_CACHE is not used: an index
means another schedule under other knob tables, and the cache's keys say which."""
import json

import torch

import paper_2004_05962_amd as bsi
import pytest
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_schedules_of_former_knob_tables_are_ignored(tmp_path, monkeypatch):
    say("batch: cache of former versions")
    dims, spac = [(40, 30, 20), (33, 21, 17)], [(5, 5, 5), (4, 4, 4)]
    path = tmp_path / "tune.json"
    monkeypatch.setenv("BSI_TUNE_CACHE", str(path))
    plan = bsi.BatchPlan(dims, spac)
    default, n = plan.config()
    grids = [torch.zeros(bsi.grid_shape(d, s), device="cuda") for d, s in zip(dims, spac)]
    fields = [torch.empty(bsi.field_shape(d), device="cuda") for d in dims]
    plan.bind(grids, fields, [torch.zeros_like(f) for f in fields], [torch.empty_like(g) for g in grids])
    plan.tune()
    plan.close()
    (key, _), = json.load(open(path)).items()
    version, rest = key.split("-", 1)
    other = (default + 1) % n
    for former in ("k1", "k2", "k3"):  # k3: its third fwd_items was 8192 items
        path.write_text(json.dumps({f"{former}-{rest}": other}))
        plan = bsi.BatchPlan(dims, spac)
        assert plan.config()[0] == default, former
        plan.close()
    path.write_text(json.dumps({f"{version}-{rest}": other}))  # this version's is
    plan = bsi.BatchPlan(dims, spac)
    assert plan.config()[0] == other
    plan.close()
