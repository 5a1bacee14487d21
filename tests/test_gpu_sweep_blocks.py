"""The recursion in one block on both sides of the layer size at which it takes
four waves or sixteen, deep graphs among them: exact costs, so values and choices
equal the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,G,shift", [(300, 1, 1, 0), (90, 11, 2, 1), (49, 16, 1, 0), (13, 31, 300, 0), (13, 32, 2, 0),
                                         (12, 33, 1, 0), (8, 41, 3, 1)])
def test_four_or_sixteen_waves(gt, orc, M, N, G, shift):
    print("[case] sweep blocks", M, N, G, shift, flush=True)
    g = np.random.default_rng(M + N)

    def costs(*shape):  # multiples of 2^-6 below 2: every sum is exact; ties and infinities
        c = (g.integers(0, 128, shape) / 64).astype(np.float32)
        return np.where(g.random(shape) < 0.2, np.float32(np.inf), c)
    Cs, Ch, Cl = costs(N), costs(M - 1, N, N), costs(N, G)
    tCh = torch.zeros(Ch.size + 1, device="cuda")[shift:][: Ch.size]
    tCh.copy_(torch.from_numpy(Ch.ravel()))
    V = torch.empty(M, N, device="cuda")
    A = torch.empty(M, N, device="cuda", dtype=torch.int32)
    Vs, a_s = torch.empty(1, device="cuda"), torch.empty(1, device="cuda", dtype=torch.int32)
    gt.gtmp_minplus_sweep(M, N, G, torch.from_numpy(Cs).cuda(), tCh, torch.from_numpy(Cl).cuda(), V, A, Vs, a_s)
    V_or, A_or, Vs_or, as_or = orc.minplus(Cs, Ch, Cl)
    assert np.array_equal(V.cpu().numpy().astype(np.float64), V_or) and np.array_equal(A.cpu().numpy(), A_or)
    assert float(Vs.item()) == Vs_or and int(a_s.item()) == as_or
