"""Restart plans with a kept stage graph past the number of graphs kept: every
call equals the plain form bit for bit and returns while earlier work on its
stream still runs, for one planner with many seeds, for more planners than are
kept (outputs of their own stand for them) and after unused graphs were
released."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

KEPT, IDLE = 64, 256


class _Busy:
    """Work on the current stream that outlasts a call's host side many times over."""

    def __init__(self):
        self.x = torch.rand((8192, 8192), device="cuda")
        self.y = torch.empty_like(self.x)
        torch.mm(self.x, self.x, out=self.y)
        torch.cuda.synchronize()

    def start(self):
        for _ in range(20):
            torch.mm(self.x, self.x, out=self.y)
        ev = torch.cuda.Event()
        ev.record()
        return ev


def _planner(gt, use_graph):
    w = wl.make_workload("2d-small", 0, M=3, N=24, H=6)
    return gt.AnytimePlanner(w, gt.GTMP_ANYTIME_RESTART, 2, use_graph=use_graph)


def _result(ap):
    return [x.clone() for x in (ap.best_cost, ap.best_meta, ap.stage_costs)]


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def test_many_seeds(gt):
    plain, ap, busy = _planner(gt, False), _planner(gt, True), _Busy()
    ap.run(0)
    for seed in range(KEPT + 12):
        print("[case] restart seed", seed, flush=True)
        ev = busy.start() if seed in (1, KEPT + 5, KEPT + 11) else None
        ap.run((seed << 32) + seed)
        assert ev is None or not ev.query()  # returned before the work ahead of it
        plain.run((seed << 32) + seed)
        assert _same(_result(ap), _result(plain)), seed


def test_more_planners_than_graphs_kept(gt):
    plain, ap, busy = _planner(gt, False), _planner(gt, True), _Busy()
    costs = [torch.empty_like(ap.stage_costs) for _ in range(KEPT + 16)]
    order = list(range(KEPT + 16)) + [0, KEPT + 15] + [KEPT + 3 + i % 4 for i in range(IDLE + 40)] + [1, KEPT + 4]
    for n, k in enumerate(order):
        print("[case] restart store call", n, "planner", k, flush=True)
        ap.stage_costs = costs[k]
        ev = busy.start() if n in (KEPT + 8, KEPT + 16, len(order) - 2, len(order) - 1) else None
        ap.run(n)
        assert ev is None or not ev.query()
        if n % 16 == 0 or ev is not None or n > len(order) - 40:
            plain.run(n)
            assert _same(_result(ap), _result(plain)), n
