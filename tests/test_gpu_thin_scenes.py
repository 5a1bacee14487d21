"""Arms of spheres without radius (or hardly any) among point obstacles, scenes
far smaller than a bin of the arm's reach: an obstacle at the very centre that the
full test forms is in contact, and the bins have to list it, for spheres on the
link and off its ends, as an edge's state and as a vertex."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_kinematics_rounding import F, _cases, _centre, _statuses

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radius", [0.0, 1e-7])
@pytest.mark.parametrize("off_link", [0.0, 1.0, 4.0])
def test_point_obstacle_at_the_centre(gt, radius, off_link):
    g = np.random.default_rng(int(10 * off_link) + (radius > 0))
    for i, joints, link, dh, t, u, v, x, _ in _cases(32):
        print("[case] thin scene", radius, off_link, i, flush=True)
        t = F(t + g.uniform(-off_link, off_link))
        c = _centre(dh, link, t, x)
        lo, hi = wl.box_limits("arm", joints)
        w = wl.make_workload("arm7", 0, M=1, N=1, H=3)
        w.update(d=joints, dh=dh, sph_link=np.array([link], np.int32), sph_t=np.array([t], F),
                 sph_r=np.array([radius], F), obs_spheres=np.array([[*c, 0.0]], F), obs_boxes=np.zeros((0, 6), F),
                 lo=lo, hi=hi, q0=u, goals=u.reshape(1, joints))
        got = _statuses(gt, w, v, x)
        assert all(s == 1 for s in got.values()), (i, got)
