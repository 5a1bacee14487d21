"""Kept graphs hold nothing of their callers' memory: a batch whose workspace
was overwritten between two calls (as after being freed and allocated again at
the same address) and a restart plan whose scene, robot or outputs changed
while its workspace, samples' key and stream stayed."""
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


@pytest.mark.parametrize("name", ["2d-small", "arm7"])
def test_restart_graph_follows_scene_robot_and_outputs(gt, name):
    print("[case] kept restart graph", name, flush=True)

    def fresh(w):
        ap = gt.AnytimePlanner(w, gt.GTMP_ANYTIME_RESTART, 3, use_graph=False)
        ap.run(5)
        return ap
    w = wl.make_workload(name, 0, M=3, N=48)
    other = wl.make_workload(name, 3, M=3, N=48)
    ap = gt.AnytimePlanner(w, gt.GTMP_ANYTIME_RESTART, 3, use_graph=True)
    ap.run(5)
    assert torch.equal(ap.stage_costs, fresh(w).stage_costs)
    # another scene (and robot), the start and goal written over in place
    keep = ap.scene  # alive, so that a graph of the first call would read valid memory
    ap.robot, ap.scene = gt.model_of(other)
    ap.q0.copy_(torch.from_numpy(other["q0"]))
    ap.goals.copy_(torch.from_numpy(other["goals"]))
    ap.run(5)
    assert torch.equal(ap.stage_costs, fresh(other).stage_costs)
    # other outputs
    old = ap.stage_costs
    ap.stage_costs = torch.full_like(old, float("nan"))
    ap.run(5)
    assert torch.equal(ap.stage_costs, old) and keep is not None
