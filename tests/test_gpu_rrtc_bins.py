"""RRT-Connect repair of arms through the obstacle bins against the general
state test: the repair takes the bins (one, two or three mask words; beyond 96
obstacles the general test), `local_path` runs the same call with the general
test, so every outcome and cost must be equal bit for bit.  Sizes: the edges of
the mask words, five spheres and 64, three joints and eight, spheres
of several radii, and trees larger than the pool a wave starts with (such calls
run again with room for both trees)."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

#        joints, spheres, obstacles (spheres, boxes), radii, (budget, cap, step, resolution, ell)
CASES = [(7, 40, (15, 15), 1, (60, 512, 0.4, 0.1, 1.5)),
         (7, 40, (16, 16), 3, (40, 64, 0.4, 0.1, 1.5)),    # 32: one word full
         (6, 33, (33, 0), 1, (40, 128, 0.4, 0.05, 1.5)),   # 33: a second word
         (7, 40, (0, 65), 2, (30, 128, 0.4, 0.1, 1.5)),    # 65: a third word
         (8, 64, (48, 48), 1, (30, 128, 0.4, 0.1, 1.5)),   # 96: three words full
         (7, 40, (49, 48), 1, (30, 128, 0.4, 0.1, 1.5)),   # 97: the general test
         (3, 5, (15, 15), 1, (40, 2, 0.5, 0.007, 1.5)),    # 72 states a segment, trees of two nodes
         (7, 40, (15, 15), 1, (1000, 512, 0.1, 0.03, 1.5))]  # trees beyond the first pool


@pytest.mark.parametrize("joints,spheres,obs,radii,lp", CASES)
def test_repair_equals_single_calls(gt, joints, spheres, obs, radii, lp):
    print("[case] rrtc bins", joints, spheres, obs, radii, lp, flush=True)
    w = wl.make_workload("arm7", 1, M=3, N=24, H=16)
    dh, sl, st, sr = wl.arm_robot(3, joints, spheres)
    sr = (sr * (1 + 0.3 * (np.arange(spheres) % radii))).astype(np.float32)
    many = sum(obs) > 40
    os_, ob = wl.arm_obstacles(5, *obs)
    if many:  # keep part of the space free
        os_[:, 3:] *= 0.4
        ob[:, 3:] *= 0.4
    lo, hi = wl.box_limits("arm", joints)
    q0, qg = wl.arm_start_goal(5, 0, joints)
    w.update(d=joints, dh=dh, sph_link=sl, sph_t=st, sph_r=sr, obs_spheres=os_, obs_boxes=ob, lo=lo, hi=hi, q0=q0,
             goals=qg.reshape(1, joints))
    stats = torch.zeros(6, device="cuda", dtype=torch.int64)
    budget, cap, step, res, ell = lp
    pl = gt.Planner(w, flags=True)
    pl.sample(w["seed"], 0)
    pl.check()
    before = pl.flags.cpu().numpy()
    pl.repair(gt.make_rrtc_opts(budget, cap, step, res, ell, stats), 9, 2)
    flags = pl.flags.cpu().numpy()
    cost = torch.cat([pl.C_s.ravel(), pl.C_h.ravel(), pl.C_l.ravel()]).cpu().numpy()
    calls, wins, _, nodes = (int(x) for x in stats.cpu().numpy()[:4])
    print("[case] calls", calls, "repaired", wins, "nodes per call", nodes / max(calls, 1), flush=True)
    assert set(np.unique(flags)) <= {0, 1, 2} and int((flags == 2).sum()) == wins and calls > 0
    assert ((flags == 0) == (before == 0)).all()
    if step == 0.1:
        assert nodes > 215 * calls  # the mean is above a first pool: some calls run again
    opts = gt.make_rrtc_opts(budget, cap, step, res, ell)
    done, failed = np.flatnonzero(flags == 2), np.flatnonzero(flags == 1)
    for e in list(done[:: max(1, len(done) // 20)]) + list(failed[:: max(1, len(failed) // 20)]):
        path, c = pl.local_path(int(e), opts, 9, 2)
        if flags[e] == 2:
            assert np.float32(c) == cost[e] and path.shape[0] >= 2, int(e)
        elif c != np.inf:  # an end point collides: the repair made no call
            u, v = _ends(w, pl, int(e))
            coll = torch.empty(2, device="cuda", dtype=torch.uint8)
            gt.gtmp_state_check(pl.robot, pl.scene, pl.d, torch.stack([u, v]).contiguous(), None, coll)
            assert int(coll.max().item()) == 1, int(e)


def _ends(w, pl, e):
    M, N = pl.M, pl.N
    if e < N:
        return pl.q0, pl.Q[0, e]
    e -= N
    if e < (M - 1) * N * N:
        m, uv = divmod(e, N * N)
        return pl.Q[m, uv // N], pl.Q[m + 1, uv % N]
    return pl.Q[M - 1, e - (M - 1) * N * N], pl.goals[0]
