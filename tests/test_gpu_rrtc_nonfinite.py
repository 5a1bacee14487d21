"""RRT-Connect repair of arms among obstacles with entries that are not numbers
or infinite (unused rows of a scene): through the obstacle bins every call is the
one `local_path` makes by the general test, and obstacles that touch nothing
there (spheres that are not numbers, obstacles at infinity) change no call."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

NAN, INF = float("nan"), float("inf")
SPHERES = {
    "radius": [[0.3, 0.2, 0.4, NAN]],
    "one coordinate": [[NAN, 0.2, 0.4, 0.2], [0.1, NAN, 0.2, 0.2], [0.3, 0.1, NAN, 0.2]],
    "whole rows": [[NAN] * 4] * 3,
    "at infinity": [[INF, 0.0, 0.0, 0.1], [0.0, -INF, INF, 0.3]],
}


def _repair(gt, w, clean=None):
    pl = gt.Planner(w, flags=True)
    pl.sample(w["seed"], 0)
    pl.check()
    if clean is not None:  # the edges to repair are those of the clean scene
        for name in ("C_s", "C_h", "C_l", "flags"):
            getattr(pl, name).copy_(getattr(clean, name))
    before = [x.clone() for x in (pl.C_s, pl.C_h, pl.C_l, pl.flags)]
    opts = gt.make_rrtc_opts(40, 128, 0.4, 0.1, 1.5)
    pl.repair(opts, 9, 2)
    return pl, before, opts


def _workload(extra_spheres=(), extra_boxes=()):
    w = wl.make_workload("arm7", 1, M=3, N=16, H=12)
    w["obs_spheres"] = np.concatenate([w["obs_spheres"], np.array(extra_spheres, np.float32).reshape(-1, 4)])
    w["obs_boxes"] = np.concatenate([w["obs_boxes"], np.array(extra_boxes, np.float32).reshape(-1, 6)])
    return w


@pytest.mark.parametrize("name", sorted(SPHERES))
def test_spheres_that_touch_nothing(gt, name):
    print("[case] rrtc spheres", name, flush=True)
    clean, before, _ = _repair(gt, _workload())
    for x, y in zip((clean.C_s, clean.C_h, clean.C_l, clean.flags), before):  # as before the repair
        y_now = x.clone()
        x.copy_(y)
        y.copy_(y_now)
    pl, _, _ = _repair(gt, _workload(SPHERES[name]), clean)
    assert int((before[3] == 2).sum().item()) > 0  # some calls succeeded
    for x, y in zip((pl.C_s, pl.C_h, pl.C_l, pl.flags), before):
        assert torch.equal(x, y)


@pytest.mark.parametrize("box", [[NAN, 0.0, 5.0, 0.1, 0.1, 0.1], [0.2, 0.3, NAN, 0.1, 0.1, NAN],
                                 [INF, 0.0, 0.0, 0.1, 0.2, 0.1], [0.0, 3.0, 3.0, INF, 0.1, 0.1]])
def test_boxes_as_in_the_general_test(gt, box):
    print("[case] rrtc box", box, flush=True)
    clean, before, _ = _repair(gt, _workload())
    for x, y in zip((clean.C_s, clean.C_h, clean.C_l, clean.flags), before):
        x.copy_(y)
    pl, _, opts = _repair(gt, _workload((), [box]), clean)
    cost = torch.cat([pl.C_s.ravel(), pl.C_h.ravel(), pl.C_l.ravel()]).cpu().numpy()
    flags = pl.flags.cpu().numpy()
    done, failed = np.flatnonzero(flags == 2), np.flatnonzero(flags == 1)
    for e in list(done[:: max(1, len(done) // 20)]) + list(failed[:: max(1, len(failed) // 20)]):
        path, c = pl.local_path(int(e), opts, 9, 2)
        if flags[e] == 2:
            assert np.float32(c) == cost[e], int(e)
        elif c != np.inf:  # an end point collides: the repair made no call
            coll = torch.empty(2, device="cuda", dtype=torch.uint8)
            ends = torch.stack([path[0], path[-1]]).contiguous()
            gt.gtmp_state_check(pl.robot, pl.scene, pl.d, ends, None, coll)
            assert int(coll.max().item()) == 1, int(e)
