"""Plans near the sizes where the launches change shape: the recursion in one
block (exact costs, so values and choices equal the oracle's: rows of one column
to a block's full width, the largest stage, one layer, several goals, costs off
a 16-byte boundary) and edge checks whose tiles are handed out by wave id (a
wave for every tile) against the same check with fewer waves than tiles."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,G,shift", [(5, 1, 1, 0), (4, 2, 2, 0), (4, 63, 1, 0), (4, 64, 1, 1), (3, 65, 3, 0),
                                         (2, 110, 1, 0), (13, 32, 1, 0), (1, 1024, 2, 0), (1, 1000, 1, 0)])
def test_recursion_in_one_block(gt, orc, M, N, G, shift):
    print("[case] one block", M, N, G, shift, flush=True)
    g = np.random.default_rng(M * N)

    def costs(*shape):  # multiples of 2^-6 below 16: every sum is exact; ties and infinities
        c = (g.integers(0, 1024, shape) / 64).astype(np.float32)
        return np.where(g.random(shape) < 0.2, np.float32(np.inf), c)
    Cs, Ch, Cl = costs(N), costs(max(M - 1, 1), N, N)[: M - 1], costs(N, G)
    tCh = torch.zeros(Ch.size + 1, device="cuda")[shift:][: Ch.size]
    tCh.copy_(torch.from_numpy(Ch.ravel()))
    V = torch.empty(M, N, device="cuda")
    A = torch.empty(M, N, device="cuda", dtype=torch.int32)
    Vs, a_s = torch.empty(1, device="cuda"), torch.empty(1, device="cuda", dtype=torch.int32)
    gt.gtmp_minplus_sweep(M, N, G, torch.from_numpy(Cs).cuda(), tCh if M > 1 else None, torch.from_numpy(Cl).cuda(), V,
                          A, Vs, a_s)
    V_or, A_or, Vs_or, as_or = orc.minplus(Cs, Ch, Cl)
    assert np.array_equal(V.cpu().numpy().astype(np.float64), V_or) and np.array_equal(A.cpu().numpy(), A_or)
    assert float(Vs.item()) == Vs_or and int(a_s.item()) == as_or


@pytest.mark.parametrize("name,M,N,G", [("2d-small", 2, 3, 1), ("2d-small", 5, 252, 1), ("2d-small", 5, 256, 3),
                                        ("arm7", 2, 5, 2), ("arm7", 5, 256, 1)])
def test_tiles_by_wave_id(gt, name, M, N, G):
    w = wl.make_workload(name, 2, M=M, N=N, H=10)
    if G > 1:
        g = np.random.default_rng(N)
        w["goals"] = np.concatenate([w["goals"], g.uniform(w["lo"], w["hi"], (G - 1, w["d"])).astype(np.float32)])
        w["G"] = G
    out = []
    for per_cu in (1, 8):  # 1024 waves and 8192 on 256 CUs; tiles: a row of up to 256 columns each
        print("[case] tiles", name, M, N, G, "blocks per CU", per_cu, flush=True)
        pl = gt.Planner(w, flags=True)
        pl.opts.blocks_per_cu = per_cu
        pl.sample(w["seed"], 0)
        pl.check()
        cost = torch.cat([pl.C_s.ravel(), pl.C_h[: M - 1].ravel(), pl.C_l.ravel()]).cpu().numpy()
        out.append((cost.view(np.uint32), pl.flags.cpu().numpy(), pl.stats[:2].cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert out[0][2][0] > 0
