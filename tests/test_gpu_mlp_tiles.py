"""BF16 inference at the edges of its tiles (16 samples, 16 outputs, 4096 tiles in
one sweep of the chip), and the descriptors at the edges of their chunks (16
neighbours of an atom, 128 slots).

Tolerances: BF16 forward 2e-2 of the result scale (8-bit mantissas on inputs,
weights and activations), the scale being at least 4: an output is a sum of 128
terms of about 0.2, of standard deviation 2, so a single one may be near zero.
Descriptors 2e-6 of max(1, value): FP64 arithmetic rounded to FP32 on both sides.
"""
import sys

import numpy as np
import pytest
import torch

import synth
from oracle import mlp as OM

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def bsm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm


@pytest.fixture(scope="module")
def ctx(bsm):
    return bsm.Context(0)


@pytest.mark.parametrize("n,M", [(1, 1), (15, 16), (16, 17), (17, 33), (250, 49), (4095, 64), (4097, 81),
                                 (65536, 97), (65537, 128)])
def test_bf16_forward_at_edges(bsm, ctx, n, M):
    say(f"bf16 forward n={n} M={M}")
    sh = OM.Shape(width=128, out_dim=M)
    rng = np.random.default_rng(n + M)
    p = (0.2 * rng.standard_normal(sh.count)).astype(np.float32)
    X = rng.uniform(-1, 1, (n, 32)).astype(np.float32)
    net = bsm.MLP(ctx, M, p)
    got = net.forward(torch.tensor(X, device=ctx.device), bsm.BF16).cpu().numpy()
    want = OM.forward(p.astype(np.float64), sh, X.astype(np.float64))
    assert got.shape == want.shape
    assert np.abs(got - want).max() < 2e-2 * max(np.abs(want).max(), 4.0)
    # samples do not depend on their tile: the last ones alone give the same bits
    k = min(n, 5)
    again = net.forward(torch.tensor(X[n - k:], device=ctx.device), bsm.BF16).cpu().numpy()
    assert np.array_equal(again, got[n - k:])
    net.close()


# rows of 5 slots (the fewest with four neighbours), 43 to 47 and 167 to 171; 1080, 9850 and 3634 slots
@pytest.mark.parametrize("rn,rc", [(2.9, 3.0), (6.0, 6.0), (10.0, 4.0)])
def test_descriptors_at_edges(bsm, ctx, rn, rc):
    say(f"descriptors rows {rn} A, slots {rc} A")
    sy = synth.displaced_frame((3, 3, 3), 4, seed=10007)
    pos = torch.tensor(sy.positions, dtype=torch.float64, device=ctx.device)
    PN = bsm.Pattern(ctx, pos, sy.box, rn, 4)
    P = bsm.Pattern(ctx, pos, sy.box, rc, 4)
    X = bsm.pair_descriptors(PN, P).cpu().numpy()
    rp, c = P.to_host()
    rows = np.repeat(np.arange(P.natoms), np.diff(rp))
    want = OM.pair_descriptors(sy.positions, sy.box, rows, c, rc, OM.atom_frames(sy.positions, sy.box, rn))
    assert X.shape == want.shape
    assert (np.abs(X - want) < 2e-6 * np.maximum(1.0, np.abs(want))).all()
    P.close()
    PN.close()
