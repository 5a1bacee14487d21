"""The two kernels that check a lazy round's list, each made to take one: a first
round of every edge between free vertices, on the side of the list's limit that
is asserted, for every kind of model behind the lists (arms among one and two
words of obstacles, more than the bins hold, spheres of one and several radii, few
spheres; points), bit for bit as the full check has it."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

BINS, OTHER = 1 << 22, 1 << 19  # (edge, state) pairs up to which the states go side by side


def _arm(N, M, obs, radii, spheres):
    w = wl.make_workload("arm7", 1, M=M, N=N, H=18)
    dh, sl, st, sr = wl.arm_robot(3, 7, spheres)
    sr = (sr * (1 + 0.3 * (np.arange(spheres) % radii))).astype(np.float32)
    os_, ob = wl.arm_obstacles(5, *obs)
    os_[:, 3:] *= 0.3  # most vertices free
    ob[:, 3:] *= 0.3
    w.update(dh=dh, sph_link=sl, sph_t=st, sph_r=sr, obs_spheres=os_, obs_boxes=ob)
    return w


CASES = [("arm, one word", BINS, lambda N, M: _arm(N, M, (15, 15), 1, 40)),
         ("arm, one word, several radii", BINS, lambda N, M: _arm(N, M, (15, 15), 3, 40)),
         ("arm, two words", BINS, lambda N, M: _arm(N, M, (30, 20), 1, 40)),
         ("arm, two words, several radii", BINS, lambda N, M: _arm(N, M, (30, 34), 3, 40)),
         ("arm, few spheres", BINS, lambda N, M: _arm(N, M, (15, 15), 1, 9)),
         ("arm, past the bins", OTHER, lambda N, M: _arm(N, M, (40, 30), 1, 40)),
         ("arm, past the bins, several radii", OTHER, lambda N, M: _arm(N, M, (40, 30), 2, 17)),
         ("points in the plane", OTHER, lambda N, M: wl.make_workload("2d-small", 1, N=N, M=M, H=18)),
         ("points in space", OTHER, lambda N, M: wl.make_workload("3d-point", 1, N=N, M=M, H=18))]


@pytest.mark.parametrize("name,limit,make", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("long", [False, True])
def test_first_round_equals_full_check(gt, name, limit, make, long):
    N = 1100 if limit == BINS else 400
    w = make(N if long else 120, 3)
    print("[case] lazy lists", name, "long" if long else "short", flush=True)
    pl = gt.Planner(w, flags=True)
    stats = torch.zeros(2, device="cuda", dtype=torch.int64)
    pl.plan_lazy(w["seed"], 0, band=1e6, max_rounds=1, stats=stats)
    pairs = int(stats[1].item()) * (w["H"] - 2)
    print("[case] pairs", pairs, "limit", limit, flush=True)
    assert pairs > limit if long else 0 < pairs <= limit
    full = gt.Planner(w, flags=True)
    full.sample(w["seed"], 0)
    full.check()
    assert torch.equal(pl.flags, full.flags)
    for a, b in ((pl.C_s, full.C_s), (pl.C_h, full.C_h), (pl.C_l, full.C_l)):
        assert torch.equal(a, b)
