"""Arms on both sides of the rule that looks their spheres up by group or by
sphere (pairs that save six lookups or seven, spheres just near enough to pair and
just too far, links no obstacle reaches), against the full test of every sphere
and obstacle: edge statuses, costs and states evaluated equal bit for bit, alone
and in a batch of both kinds."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

R = 0.05


def _link(link, n, gap, length):
    """n spheres of a link, `gap` radii apart."""
    return [(link, float(gap * R * i / length)) for i in range(n)]


def _workload(spheres, joints, obs, radii, far=False):
    w = wl.make_workload("arm7", 1, M=3, N=72, H=18)
    dh, _, _, _ = wl.arm_robot(4, joints, 8)
    length = np.hypot(dh[:, 0], dh[:, 2])
    s = [x for link, n, gap in spheres for x in _link(link, n, gap, length[link - 1])]
    os_, ob = wl.arm_obstacles(6, *obs)
    os_[:, 3:] *= 0.5
    ob[:, 3:] *= 0.5
    if far:  # nothing within reach of the first links
        os_[:, :3] += 1.2 * os_[:, :3] / np.linalg.norm(os_[:, :3], axis=1, keepdims=True)
        ob[:, :3] += 1.2 * ob[:, :3] / np.linalg.norm(ob[:, :3], axis=1, keepdims=True)
    lo, hi = wl.box_limits("arm", joints)
    q0, qg = wl.arm_start_goal(5, 0, joints)
    n = len(s)
    w.update(d=joints, dh=dh, sph_link=np.array([x[0] for x in s], np.int32), sph_t=np.array([x[1] for x in s], np.float32),
             sph_r=(R * (1 + 0.3 * (np.arange(n) % radii))).astype(np.float32), obs_spheres=os_.astype(np.float32),
             obs_boxes=ob.astype(np.float32), lo=lo, hi=hi, q0=q0, goals=qg.reshape(1, joints))
    return w


CASES = {  # (link, spheres, radii apart), joints, radii
    "one sphere": ([(7, 1, 1.0)], 7, 1),
    "six saved": ([(3, 6, 2.4), (6, 7, 2.4)], 7, 1),
    "seven saved": ([(3, 6, 2.4), (6, 9, 2.4)], 7, 1),
    "seven saved, five groups a link": ([(4, 10, 1.0), (5, 5, 1.0), (6, 1, 1.0)], 6, 1),
    "just apart": ([(2, 7, 2.6), (4, 8, 2.6), (5, 5, 2.6)], 5, 1),
    "several radii": ([(2, 9, 1.5), (4, 8, 4.0)], 4, 3),
}


@pytest.mark.parametrize("obs", [(18, 14), (30, 30)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_lookups_equal_full_test(gt, name, obs):
    spheres, joints, radii = CASES[name]
    for far in (False, True):
        w = _workload(spheres, joints, obs, radii, far)
        out = []
        for chunks in (0, 2):
            print("[case] sphere lookups", name, obs, far, chunks, flush=True)
            pl = gt.Planner(w, flags=True)
            pl.opts.sphere_chunks = chunks
            pl.plan(w["seed"], 0)
            cost = torch.cat([pl.C_s.ravel(), pl.C_h[: pl.M - 1].ravel(), pl.C_l.ravel()]).cpu().numpy()
            out.append((cost.view(np.uint32), pl.flags.cpu().numpy(), int(pl.stats[0].item())))
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]
        assert 0 < int((out[0][1] == 0).sum())


@pytest.mark.parametrize("names", [("one sphere", "six saved", "just apart"), tuple(sorted(CASES))])
@pytest.mark.parametrize("obs", [(18, 14), (30, 30)])
def test_batch_equals_single(gt, names, obs):
    print("[case] sphere lookups batch", names, obs, flush=True)
    ws = [_workload(CASES[n][0], CASES[n][1], obs, CASES[n][2]) for n in names]
    bp = gt.BatchPlanner([dict(w=w, mode="plain", seed=40 + i) for i, w in enumerate(ws)], use_graph=False)
    bp.run()
    for i, w in enumerate(ws):
        pl = gt.Planner(w)
        pl.plan(40 + i, 0)
        assert torch.equal(bp.best_cost[i], pl.cost[0]), names[i]
