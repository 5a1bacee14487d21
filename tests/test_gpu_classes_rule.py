"""The class sweep against the sequential list rule of its definition (a
successor at a time, in index order; a full list keeps the cheapest), written
out in Python with FP32 sums: the same labels, costs, chains and count of
dropped labels.  Sizes around the runs of successors a vertex is split into,
lists that never fill, fill and overflow, several goals, and the archive past
its capacity."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def _edge_label(u, v, reps):
    out = []
    for z in reps:
        f = np.float32
        if (u[0] < z[0]) == (v[0] < z[0]):
            out.append(0)
            continue
        dx, dy, ex, ey = f(v[0] - u[0]), f(v[1] - u[1]), f(z[0] - u[0]), f(z[1] - u[1])
        cr = f(f(dx * ey) - f(dy * ex))
        above = cr < 0 if dx > 0 else cr > 0
        out.append((1 if dx > 0 else -1) if above else 0)
    return np.array(out)


def _build(u, succ, costs, lists, reps, L, penalty):
    """One vertex's list and its dropped labels."""
    ent, dropped = [], 0
    for v, c in enumerate(costs):
        if not c < penalty:
            continue
        kap = _edge_label(u, succ[v], reps)
        src = lists[v] if lists is not None else [(tuple([0] * len(reps)), None, None)]
        cand = [(tuple(kap + np.array(lab)), c if j is None else np.float32(c + j), (v, e))
                for e, (lab, j, _) in enumerate(src)]
        known = {lab: i for i, (lab, _, _) in enumerate(ent)}
        new = []
        for lab, cc, nx in cand:
            if lab in known:
                if cc < ent[known[lab]][1]:
                    ent[known[lab]] = (lab, cc, nx)
            else:
                new.append((lab, cc, nx))
        for x in new:
            if len(ent) < L:
                ent.append(x)
                continue
            dropped += 1
            worst = max(range(len(ent)), key=lambda i: (ent[i][1], i))
            if x[1] < ent[worst][1]:
                ent[worst] = x
    return ent, dropped


@pytest.mark.parametrize("scene,N,M,G,L", [(0, 7, 2, 1, 64), (1, 9, 4, 3, 64), (2, 64, 3, 1, 4), (1, 65, 4, 2, 16),
                                           (3, 33, 1, 5, 2), (4, 70, 3, 1, 1), (0, 80, 6, 1, 64)])
def test_sweep_follows_the_list_rule(gt, scene, N, M, G, L):
    print("[case] class rule", scene, N, M, G, L, flush=True)
    w = wl.make_workload("2d-small", scene, N=N, M=M)
    if G > 1:
        g = np.random.default_rng(G)
        w["goals"], w["G"] = np.concatenate([w["goals"], g.uniform(-9, 9, (G - 1, 2)).astype(np.float32)]), G
    reps = w["circles"][:, :2]
    pl = gt.Planner(w)
    pl.plan(w["seed"], 0)
    got, ovf = gt.class_sweep(pl, reps, L=L)
    Q, Cs, Ch, Cl = (x.cpu().numpy() for x in (pl.Q, pl.C_s, pl.C_h, pl.C_l))
    lists, total = None, 0
    for m in range(M - 1, -1, -1):
        rows = [_build(Q[m, u], w["goals"] if m == M - 1 else Q[m + 1], Cl[u] if m == M - 1 else Ch[m, u],
                       None if m == M - 1 else below, reps, L, w["penalty"]) for u in range(N)]
        below = [r[0] for r in rows]
        total += sum(r[1] for r in rows)
        lists = [below] + (lists or [])
    start, d = _build(w["q0"], Q[0], Cs, lists[0], reps, L, w["penalty"])
    total += d
    print("[case] classes", len(start), "dropped", total, flush=True)
    assert ovf == total and set(got) == {lab for lab, _, _ in start}
    for lab, cost, nx in start:
        chain, n = [], nx
        for m in range(M):
            chain.append(n[0])
            n = lists[m][n[0]][n[1]][2]
        chain.append(n[0])
        assert np.float32(got[lab][0]) == cost and got[lab][1] == chain


def test_archive_capacity(gt):
    """Past its capacity the archive keeps the first classes met, in class
    order, and counts the others."""
    w = wl.make_workload("2d-small", 0, N=48, M=4)
    reps = w["circles"][:, :2]
    full = gt.ClassPlanner(w, reps, 4, L=64, cap=1024)
    full.run(w["seed"])
    n, base = int(full.a_count.item()), int(full.overflow.item())
    cap = max(1, n - 3)
    small = gt.ClassPlanner(w, reps, 4, L=64, cap=cap)
    small.run(w["seed"])
    print("[case] archive", n, "capacity", cap, flush=True)
    assert int(small.a_count.item()) == min(n, cap)
    assert torch.equal(small.a_lab, full.a_lab[:cap]) and torch.equal(small.a_cost, full.a_cost[:cap])
    assert int(small.overflow.item()) - base >= n - cap
