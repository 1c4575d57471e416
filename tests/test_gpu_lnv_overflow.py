"""An LNV step whose energy leaves FP64's range says so and leaves L's bits.

Eight atoms too far apart to meet (b = 4, S = 1).  Seven have L = 0.3, H = h and a zero block
of Z, so that their part of the preconditioned gradient, and with it the direction, is exactly
zero and the line search is the eighth atom's alone.  With h = 1 the step succeeds.  With
h = 2e307, 3 Tr XY - 2 Tr WY = 6.048 h is still in range and E, twice that, is not.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm


def step(bsm, h, mode):
    ctx = bsm.Context(0)
    pos = np.stack(np.meshgrid(*[[0.0, 4.0]] * 3, indexing="ij"), -1).reshape(-1, 3)
    P = bsm.Pattern(ctx, pos, (8.0, 8.0, 8.0), 2.0, 4)
    assert P.nnzb == 8
    one = np.broadcast_to(np.eye(4), (8, 4, 4))
    H, L, Z = h * one, 0.3 * one, 0.0 * one
    Z[7] = one[7]
    H[7] = np.diag([-1.0, -0.5, 0.3, 0.8]) + 0.01
    L[7] = np.diag([0.6, 0.55, 0.4, 0.3])
    S, H, Z, L = (bsm.Matrix(P, torch.tensor(np.ascontiguousarray(m), device=ctx.device)) for m in (one, H, Z, L))
    before = L.blocks.clone()
    lnv = bsm.LNV(S, H, Z, L, 8.0, mode=mode, mu=0.1, init_from_z=False)
    r = lnv.step()
    same = torch.equal(L.blocks, before)
    lnv.close()
    ctx.close()
    return r, same


@pytest.mark.parametrize("mode", [0, 1])
def test_energy_past_the_range_leaves_L(bsm, mode):
    r, same = step(bsm, 1.0, mode)
    assert r.status == bsm.OK and not same
    r, same = step(bsm, 2e307, mode)
    assert r.status == bsm.ENONFINITE and not np.isfinite(r.E)
    assert same
