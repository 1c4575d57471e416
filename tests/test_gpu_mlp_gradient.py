"""FP32 loss gradients at the edges of their tiles (16 samples, 32 output columns),
sample ranges (up to 32 of them) and chunks (8192 samples), against the FP64 oracle.

Tolerance: 1e-5 of the largest gradient.  Sums run over at most 256 samples of a
range, 32 ranges and 2 chunks, and over 128-term products before them: some 500
FP32 roundings of 6e-8 that accumulate like their square root, 1.3e-6, and leave a
margin of 7 for the tanh of both sides and for cancellation in the sums.
"""
import sys

import numpy as np
import pytest
import torch

from oracle import mlp as OM

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm


@pytest.fixture(scope="module")
def ctx(bsm):
    return bsm.Context(0)


@pytest.mark.parametrize("n,M", [(1, 1), (15, 16), (17, 33), (64, 81), (65, 128), (2049, 64), (8192, 32),
                                 (8193, 81), (16400, 100)])
def test_gradient_at_edges(bsm, ctx, n, M):
    print(f"gradient n={n} M={M}", flush=True)
    sys.stdout.flush()
    sh = OM.Shape(width=128, out_dim=M)
    rng = np.random.default_rng(n + M)
    p = (0.2 * rng.standard_normal(sh.count)).astype(np.float32)
    X = rng.uniform(-1, 1, (n, 32)).astype(np.float32)
    T = rng.uniform(-1, 1, (n, M)).astype(np.float32)
    net = bsm.MLP(ctx, M, p)
    Xd, Td = (torch.tensor(a, device=ctx.device) for a in (X, T))
    net.loss_grad(Xd[:1] + 1, Td[:1])      # leaves other partial sums behind
    loss, g = net.loss_grad(Xd, Td)
    lo, go = OM.loss_grad(p.astype(np.float64), sh, X.astype(np.float64), T.astype(np.float64))
    assert abs(loss - lo) < 1e-5 * lo
    assert np.abs(g.cpu().numpy() - go).max() < 1e-5 * np.abs(go).max()
    # the same sums through a permuted minibatch: one plain step of the optimiser moves each weight
    # against its gradient
    perm = rng.permutation(n).astype(np.int32)
    net.train(Xd, Td, epochs=1, batch=n, lr=1e-3, perm=torch.tensor(perm, device=ctx.device))
    sure = np.abs(go) > 1e-4 * np.abs(go).max()
    moved = net.params - p
    assert np.array_equal(np.sign(moved[sure]), -np.sign(go[sure]))
    net.close()
