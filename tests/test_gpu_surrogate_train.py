"""The surrogate's training step over its batch sizes: the smallest (one slab
of rows per batch split), an odd number of slabs per split and more slabs than
CUs; gradients and loss against the FP64 oracle with the BF16 rounding points
of the network, bit-equal on repetition."""
import numpy as np
import pytest
import torch

import oracle.surrogate as OS
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(256, 7), (768, 2), (8192 + 256, 8)])
def test_gradients_over_batch_sizes(gt, n, d):
    print("[case] train", n, d, flush=True)
    P, Bf = wl.surrogate_init(11 + d, d)
    rng = np.random.default_rng([n, d])
    for k in ("b1", "b2", "b3", "b4", "b5"):
        P[k] = (0.1 * rng.standard_normal(P[k].shape)).astype(np.float32)
    X = rng.uniform(-np.pi, np.pi, (n, d)).astype(np.float32)
    y = (rng.random(n) < 0.4).astype(np.uint8)
    net = gt.Surrogate(P, Bf, batch=n)
    Xg, yg = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    z = torch.empty(n, device="cuda")
    loss = float(net.grad(Xg, yg, logits=z).item())
    g1 = net.grad_buf.clone()
    assert float(net.grad(Xg, yg).item()) == loss and torch.equal(g1, net.grad_buf)
    P64, X64 = {k: v.astype(np.float64) for k, v in P.items()}, X.astype(np.float64)
    want, G = OS.loss_and_grad(P64, OS.features(X64, Bf), y.astype(np.float64))
    # a mean of terms whose derivative in the logit is at most 1 in size
    dz = np.abs(z.cpu().numpy() - OS.logits_of_states(P64, Bf, X64))
    assert abs(loss - want) <= dz.mean() + 1e-6 * want
    g = g1.cpu().numpy().astype(np.float64)
    for i, k in enumerate(gt.SUR_NAMES):
        lo, hi = net.offsets[i], net.offsets[i + 1] if i < 9 else net.total
        ref = np.asarray(G[k], np.float64).ravel()
        rel = np.linalg.norm(g[lo:hi] - ref) / np.linalg.norm(ref)
        print("[case] grad", k, rel, flush=True)
        assert rel <= 1e-3, (k, rel)  # the bound of the other gradient tests
