"""Kept graphs hold nothing of their callers' memory: a batch whose workspace
was overwritten between two calls (as after being freed and allocated again at
the same address)."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def test_batch_workspace_overwritten_between_calls(gt):
    print("[case] kept batch graph, workspace overwritten", flush=True)
    specs = [dict(w=wl.make_workload("2d-small", 0), mode="plain"),
             dict(w=wl.make_workload("arm7", 0, N=64, M=3), mode="restart", stages=2),
             dict(w=wl.make_workload("arm7", 2, N=48, M=4), mode="growing", stages=4, M_min=3, N_min=12)]
    bp = gt.BatchPlanner(specs, use_graph=True)
    bp.best_wp.zero_()
    bp.best_idx.fill_(-1)
    want = None
    for fill in (None, 0, 255):
        if fill is not None:
            bp.workspace.fill_(fill)
        bp.run()
        got = [x.clone() for x in (bp.best_cost, bp.best_idx, bp.best_wp, bp.best_meta, bp.stage_costs)]
        want = want or got
        assert all(torch.equal(a.nan_to_num(-7.0), b.nan_to_num(-7.0)) for a, b in zip(want, got)), fill
