"""Arms through the obstacle bins, looked up by groups of one or two
neighbouring spheres, against the full test of every sphere and every obstacle
(sphere_chunks = 2): edge statuses, costs and states evaluated equal bit for
bit.  Robots: 1, 2, 8, 9, 16, 17 and all 64 spheres on one link (the edges of a
link's four groups), links without spheres, neighbours too far apart to share a
lookup, spheres off the ends of their link, several radii, two to eight joints;
one and two mask words."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def _even(*counts):
    return [(j + 1, (i + 0.5) / n) for j, n in enumerate(counts) for i in range(n)]


ROBOTS = {
    "odd counts": (7, _even(1, 2, 3, 8, 9, 7, 5), 0.05, 1),
    "long links": (4, _even(17, 16, 0, 9), 0.04, 3),
    "one link": (3, _even(0, 64, 0), 0.03, 1),
    "last link": (8, [(8, 0.5)], 0.05, 1),
    "far apart": (7, _even(2, 2, 3, 2, 3, 2, 2), 0.02, 2),
    "off the link": (6, [(L, t) for L in range(1, 7) for t in (-0.6, -0.55, 0.2, 1.0, 1.3, 1.9)], 0.05, 1),
    "two joints": (2, _even(3, 4), 0.05, 2),
}


@pytest.mark.parametrize("obs", [(18, 14), (20, 13)])  # 32 obstacles: one mask word; 33: two
@pytest.mark.parametrize("robot", sorted(ROBOTS))
def test_groups_equal_full_test(gt, robot, obs):
    joints, spheres, r, radii = ROBOTS[robot]
    w = wl.make_workload("arm7", 1, M=3, N=96, H=18)
    dh, _, _, _ = wl.arm_robot(4, joints, len(spheres))
    link = np.array([s[0] for s in spheres], np.int32)
    t = np.array([s[1] for s in spheres], np.float32)
    rad = (r * (1 + 0.4 * (np.arange(len(spheres)) % radii))).astype(np.float32)
    os_, ob = wl.arm_obstacles(6, *obs)
    os_[:, 3:] *= 0.6
    ob[:, 3:] *= 0.6
    lo, hi = wl.box_limits("arm", joints)
    q0, qg = wl.arm_start_goal(5, 0, joints)
    w.update(d=joints, dh=dh, sph_link=link, sph_t=t, sph_r=rad, obs_spheres=os_, obs_boxes=ob, lo=lo, hi=hi, q0=q0,
             goals=qg.reshape(1, joints))
    out = []
    for chunks in (0, 2):
        print("[case] sphere groups", robot, obs, "chunks", chunks, flush=True)
        pl = gt.Planner(w, flags=True)
        pl.opts.sphere_chunks = chunks
        pl.sample(w["seed"], 0)
        pl.check()
        cost = torch.cat([pl.C_s.ravel(), pl.C_h[: pl.M - 1].ravel(), pl.C_l.ravel()]).cpu().numpy()
        out.append((cost.view(np.uint32), pl.flags.cpu().numpy(), int(pl.stats[0].item())))
    (cg, fg, sg), (cd, fd, sd) = out
    print("[case] edges", fg.size, "free", int((fg == 0).sum()), "states", sg, sd, flush=True)
    assert np.array_equal(fg, fd) and np.array_equal(cg, cd) and sg == sd
    assert 0 < int((fg == 0).sum())  # an edge went through every state
