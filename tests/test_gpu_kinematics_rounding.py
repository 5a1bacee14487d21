"""The arm's kinematics are FP32 computations whose roundings are written out,
so the status of a state that touches an obstacle to the last bit is the same in
every kernel.  The centre of a sphere is formed in numpy by the same operations
(a fused multiply-add exactly, its one rounding at the end); an obstacle's radius
is then the smallest that the centre touches, and the next smaller one it does
not: every check has to find contact for the one and none for the other."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

F, LD = np.float32, np.longdouble


def _fma(a, b, c):
    return F(LD(a) * LD(b) + LD(c))


def _sincos(x):
    """As joint_sincos, |x| <= 32."""
    k = np.rint(F(x * F(0.636619772367581)))
    r = _fma(-k, F(-4.371138828673793e-08), _fma(-k, F(1.5707963705062866), x))
    z = F(r * r)
    ps = _fma(z, _fma(z, F(-1.949563593e-04), F(8.331978694e-03)), F(-1.666665077e-01))
    sr = _fma(F(r * z), ps, r)
    pc = _fma(z, _fma(z, F(-1.359782298e-03), F(4.165629297e-02)), F(-4.999989569e-01))
    cr = _fma(z, pc, F(1))
    return [(sr, cr), (cr, -sr), (-sr, -cr), (-cr, sr)][int(k) & 3]


def _sop(u, v, x, y):
    """u v + x y, the second product rounded first."""
    return _fma(u, v, F(x * y))


def _centre(dh, link, t, q):
    """Centre of the sphere at fraction t of the link (> 2), twists 0 and +-pi/2
    exact."""
    p = b = np.zeros(3, F)
    for j in range(link):
        a, al, dz, off = dh[j]
        s, c = _sincos(F(q[j] + off))
        quarter = abs(abs(float(al)) - np.pi / 2) <= 1e-7
        ca, sa = (F(1), F(0)) if al == 0 else (F(0), F(np.sign(al))) if quarter else (F(np.cos(float(al))),
                                                                                  F(np.sin(float(al))))
        if j == 0:
            x, y, z = np.array([c, s, 0], F), np.array([-F(ca * s), F(ca * c), sa], F), \
                np.array([F(sa * s), -F(sa * c), ca], F)
            b, p = p, np.array([F(a * c), F(a * s), dz], F)
            continue
        xn = np.array([_sop(s, y[i], c, x[i]) for i in range(3)], F)
        yp = np.array([_sop(c, y[i], -s, x[i]) for i in range(3)], F)
        step = [_sop(a, xn[i], dz, z[i]) for i in range(3)]
        b, p = p, np.array([F(p[i] + step[i]) for i in range(3)], F)
        if al == 0:
            y = yp
        elif quarter:
            y, z = (z, -yp) if al > 0 else (-z, yp)
        else:
            y, z = np.array([_sop(sa, z[i], ca, yp[i]) for i in range(3)], F), \
                np.array([_sop(ca, z[i], -sa, yp[i]) for i in range(3)], F)
        x = xn
    return np.array([_fma(t, F(p[i] - b[i]), b[i]) for i in range(3)], F)


def _touches(c, o, ro, r):
    R = F(F(ro) + F(r))
    g = -F(R * R)
    for i in range(3):
        dlt = F(c[i] - o[i])
        g = _fma(dlt, dlt, g)
    return g <= 0


def _radius(c, o, r):
    """The smallest obstacle radius at o that a sphere of radius r at c touches."""
    ro = F(np.sqrt(np.sum((LD(1) * c - o) ** 2)) - r)
    while _touches(c, o, ro, r):
        ro = np.nextafter(ro, F(0))
    while not _touches(c, o, ro, r):
        ro = np.nextafter(ro, F(9))
    return ro


def _cases(n):
    """An arm of one sphere and an edge u -> v whose middle state x is clear of
    both ends' sphere."""
    g = np.random.default_rng(77)
    i = 0
    while i < n:
        joints, link = (7, 7) if i % 2 else (6, 5)
        dh, _, _, _ = wl.arm_robot(100 + i, joints, 8)
        if i % 3 == 0:
            dh[:, 1] = g.uniform(-1.5, 1.5, joints)
        dh, t = dh.astype(F), F(g.uniform(0.1, 0.9))
        u, v = g.uniform(-2, 2, (2, joints)).astype(F)
        x = np.array([_fma(F(0.5), F(v[k] - u[k]), u[k]) for k in range(joints)], F)
        cu, cv, cx = (_centre(dh, link, t, q) for q in (u, v, x))
        if min(np.linalg.norm(cx - cu), np.linalg.norm(cx - cv)) < 0.2:
            continue
        yield i, joints, link, dh, t, u, v, x, g.normal(size=3)
        i += 1


def _statuses(gt, w, v, x):
    """Contact of x: as a state, as the middle state of the edge q0 -> v and as a
    vertex (by the bins and by every obstacle)."""
    d, out = w["d"], {}
    robot, scene = gt.model_of(w)
    coll = torch.empty(1, device="cuda", dtype=torch.uint8)
    gt.gtmp_state_check(robot, scene, d, torch.from_numpy(x.reshape(1, d)).cuda(), None, coll)
    out["state"] = int(coll.item())
    for name, chunks, q in (("edge, bins", 0, v), ("edge", 2, v), ("vertex, bins", 0, x), ("vertex", 2, x)):
        pl = gt.Planner(w, flags=True)
        pl.opts.sphere_chunks = chunks
        pl.Q.copy_(torch.from_numpy(q.reshape(1, 1, d)))
        pl.check()
        out[name] = int(pl.flags[0].item())
    return out


def test_contact_to_the_last_bit(gt):
    for i, joints, link, dh, t, u, v, x, way in _cases(48):
        print("[case] kinematics rounding", i, flush=True)
        r = F(0.04)
        lo, hi = wl.box_limits("arm", joints)
        c = _centre(dh, link, t, x)
        o = (c + 0.06 * way / np.linalg.norm(way)).astype(F)
        ro = _radius(c, o, r)
        for radius, want in ((ro, 1), (np.nextafter(ro, F(0)), 0)):
            w = wl.make_workload("arm7", 0, M=1, N=1, H=3)
            w.update(d=joints, dh=dh, sph_link=np.array([link], np.int32), sph_t=np.array([t], F),
                     sph_r=np.array([r], F), obs_spheres=np.array([[*o, radius]], F),
                     obs_boxes=np.zeros((0, 6), F), lo=lo, hi=hi, q0=u, goals=u.reshape(1, joints))
            got = _statuses(gt, w, v, x)
            assert all(s == want for s in got.values()), (i, want, got)
