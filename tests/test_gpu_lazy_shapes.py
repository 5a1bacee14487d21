"""Lazy plans over the shapes of their passes against the full check, bit for
bit: rows that are not a multiple of four columns, fewer samples than a block's
rows, a column past a block's segment, several goals, unaligned cost and status
arrays, one layer, and robots whose lists go either way."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,M,N,G,shift,band", [("arm7", 4, 3, 1, 0, 0.5), ("arm7", 3, 261, 2, 0, 0.3),
                                                   ("2d-small", 5, 64, 3, 0, 0.2), ("2d-small", 1, 70, 2, 0, 0.2),
                                                   ("3d-point", 3, 1028, 1, 0, 0.1), ("arm7", 3, 256, 1, 1, 2.0),
                                                   ("2d-large", 3, 1025, 1, 0, 0.05)])
def test_lazy_equals_full(gt, name, M, N, G, shift, band):
    print("[case] lazy shapes", name, M, N, G, shift, band, flush=True)
    w = wl.make_workload(name, 2, M=M, N=N)
    if G > 1:
        g = np.random.default_rng(N)
        w["goals"] = np.concatenate([w["goals"], g.uniform(w["lo"], w["hi"], (G - 1, w["d"])).astype(np.float32)])
        w["G"] = G
    full = gt.Planner(w, flags=True)
    full.plan(w["seed"], 0)
    pl = gt.Planner(w, flags=True)
    if shift:  # costs off a 16-byte boundary, statuses off a 4-byte one
        pl.C_h = torch.empty(pl.C_h.numel() + 1, device="cuda")[1:].reshape(pl.C_h.shape)
        pl.flags = torch.empty(pl.E + 1, device="cuda", dtype=torch.uint8)[1:]
    stats = torch.zeros(2, device="cuda", dtype=torch.int64)
    status, rounds = pl.plan_lazy(w["seed"], 0, band=band, stats=stats)
    assert status == gt.GTMP_OK and int(stats[0].item()) == rounds
    assert torch.equal(pl.cost, full.cost) and torch.equal(pl.wp.isnan(), full.wp.isnan())
    known = pl.flags != 0xFF
    assert torch.equal(pl.flags[known], full.flags[known])

    def flat(p):
        return torch.cat([p.C_s.ravel(), p.C_h[: M - 1].ravel(), p.C_l.ravel()])
    a, b = flat(pl), flat(full)
    assert torch.equal(a[known], b[known])
    assert bool((a <= b).all())  # unchecked costs are lower bounds
    # endpoint failures are known from the start, the rest is what the rounds checked
    print("[case] rounds", rounds, "checked", int(stats[1].item()), "known", int(known.sum().item()), flush=True)
