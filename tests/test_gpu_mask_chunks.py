"""mask_copy on both sides of the lines between its chunks of 64 and of 256 slots, onto a wider
and onto a narrower pattern: copies, so bits are equal to a gather's.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def lattice(cells, seed):
    a = 5.43
    base = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0], [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]]) * (a / 4)
    at = np.stack(np.meshgrid(*[np.arange(m) * a for m in cells], indexing="ij"), -1).reshape(-1, 1, 3)
    pos = (at + base).reshape(-1, 3)
    return pos + np.random.default_rng(seed).normal(0, 0.1, pos.shape), [a * m for m in cells]


def keys(P, device):
    rp, cols = P.to_host()
    rows = np.repeat(np.arange(P.natoms), np.diff(rp))
    return torch.tensor(rows.astype(np.int64) * P.natoms + cols, device=device)


# slots of the wider pattern: some 2^17 and 2^21 are the lines for b <= 5 and for larger b
@pytest.mark.parametrize("b,cells,wide,narrow", [(1, (2, 2, 2), 6.0, 3.0), (5, (7, 7, 7), 5.9, 4.0), (5, (8, 8, 8), 5.9, 4.0),
                                                 (4, (8, 8, 8), 7.0, 5.0), (6, (8, 8, 8), 12.9, 5.0),
                                                 (6, (8, 8, 8), 13.7, 5.0), (9, (2, 2, 3), 7.0, 5.0)])
def test_mask_copy_of_both_chunks(b, cells, wide, narrow):
    import paper_2205_08941_amd as bsm
    ctx = bsm.Context(0)
    pos, box = lattice(cells, 7)
    pos = pos[:-3]   # ragged
    W, N = bsm.Pattern(ctx, pos, box, wide, b), bsm.Pattern(ctx, pos, box, narrow, b)
    print("mask copy", b, len(pos), W.nnzb, N.nnzb, flush=True)
    kw, kn = keys(W, ctx.device), keys(N, ctx.device)
    g = torch.Generator(device=ctx.device)
    g.manual_seed(3)
    for src, dst, ks, kd in ((W, N, kw, kn), (N, W, kn, kw)):
        A = bsm.Matrix(src, torch.randn((src.nnzb, b, b), dtype=torch.float64, device=ctx.device, generator=g))
        C = bsm.Matrix(dst, torch.full((dst.nnzb, b, b), float("nan"), dtype=torch.float64, device=ctx.device))
        bsm.mask_copy(A, C)
        at = torch.searchsorted(ks, kd).clamp(max=src.nnzb - 1)
        want = torch.where((ks[at] == kd)[:, None, None], A.blocks[at], torch.zeros((), dtype=torch.float64, device=ctx.device))
        assert torch.equal(C.blocks, want)
    ctx.close()
