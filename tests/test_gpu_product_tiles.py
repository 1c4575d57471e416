"""Products at the edges of the tile choices: two-, four- and eight-row ring tiles,
direct and transposed, single and paired, and the copies of b = 4 operands that do
not start at 16-byte boundaries.  Every choice sums the same terms in the same
order, so results must equal the 8-row tiles' bit for bit; the 8-row result is held
to the oracle at 1e-12 of its scale (sums of at most a few hundred terms of order
one: rounding below 1e-13).
"""
import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsm():
    import paper_2205_08941_amd as m
    return m


@pytest.fixture()
def ctx(bsm):
    c = bsm.Context(0)
    yield c
    c.close()


def operands(bsm, ctx, cells, b, cutoffs):
    import torch
    s = synth.make_system("t", cells, 4, synth.SMALL_CUTOFFS, 11, displacement_sigma=0.1)
    g = {r: bsm.Pattern(ctx, s.positions, s.box, r, b) for r in set(cutoffs)}
    o = {r: O.create_pattern(s.positions, s.box, r) for r in set(cutoffs)}
    host = [synth.random_blocks(o[r].nnz, b, 31 + k) for k, r in enumerate(cutoffs[:2])]
    mats = [bsm.Matrix(g[r], torch.tensor(h, device=ctx.device)) for r, h in zip(cutoffs, host)]
    return g, o, host, mats


# one atom short of, at and past a row group's edge is given by 64 + 8 n atoms of cells and
# by the tile edges of each pattern; a 1 x 1 x 2 box has 16 atoms and a single column tile
@pytest.mark.parametrize("b", [4, 9])
@pytest.mark.parametrize("cells,cutoffs", [((1, 1, 2), (5.0, 5.0, 5.0)), ((2, 2, 2), (8.0, 6.0, 14.0)),
                                           ((2, 2, 3), (14.0, 8.0, 8.0)), ((2, 3, 3), (8.0, 8.0, 8.0))])
def test_rows_and_transposes_agree(bsm, ctx, b, cells, cutoffs):
    import torch
    g, o, host, (A, B) = operands(bsm, ctx, cells, b, cutoffs)
    ra, rb, rc = cutoffs
    for alpha, beta in ((1.0, 0.0), (-0.7, 0.3)):
        c0 = synth.random_blocks(o[rc].nnz, b, 47)
        ref = O.Matrix(o[rc], b, c0.copy())
        O.multiply_truncate(alpha, O.Matrix(o[ra], b, host[0]), O.Matrix(o[rb], b, host[1]), beta, ref)
        first = None
        for rows, tmode in ((8, 0), (8, 2), (4, 0), (4, 2), (2, 0), (2, 2), (0, 1)):
            ctx.set_rows_per_wave(rows)
            ctx.set_transposed_plans(tmode)
            print("product tiles", b, cells, cutoffs, rows, tmode, beta, flush=True)
            C = bsm.Matrix(g[rc], torch.tensor(c0, device=ctx.device))
            bsm.multiply_truncate(alpha, A, B, beta, C)
            got = C.blocks.cpu().numpy()
            if first is None:
                first = got
                assert np.abs(got - ref.blocks).max() <= 1e-12 * np.abs(ref.blocks).max()
            assert np.array_equal(got, first), (rows, tmode)


@pytest.mark.parametrize("offset", [0, 1])
def test_packed_copies_need_no_alignment(bsm, ctx, offset):
    """b = 4 operands one element past a 16-byte boundary take the 4-byte copies: same bits."""
    import torch
    g, o, host, (A, B) = operands(bsm, ctx, (2, 2, 2), 4, (8.0, 6.0, 14.0))
    C, D = bsm.Matrix(g[14.0]), bsm.Matrix(g[14.0])
    bsm.multiply_truncate(1.0, A, B, 0.0, C)
    moved = []
    for M in (A, B):
        buf = torch.empty(M.blocks.numel() + 2, dtype=torch.float64, device=ctx.device)
        v = buf[offset:offset + M.blocks.numel()].view(M.blocks.shape)
        v.copy_(M.blocks)
        moved.append(bsm.Matrix(M.pattern, v))
    bsm.multiply_truncate(1.0, moved[0], moved[1], 0.0, D)
    assert torch.equal(C.blocks, D.blocks)
    bsm.multiply_truncate_pair(1.0, moved[0], A, moved[1], 0.0, C, D)
    assert torch.equal(C.blocks, D.blocks)


@pytest.mark.parametrize("b", [5, 6, 7, 8, 10, 11, 12, 13, 14, 15, 16])
def test_ring_of_other_block_sizes(bsm, ctx, b):
    """The ring kernels of the other block sizes against the scalar-operand kernel (variant 0),
    which sums the same terms in the same order, and against the oracle; a non-finite A block
    reaches exactly the output blocks of its own triples."""
    import torch
    cutoffs = (8.0, 6.0, 10.0)
    g, o, host, (A, B) = operands(bsm, ctx, (2, 2, 3), b, cutoffs)
    ref = O.Matrix(o[10.0], b, np.zeros((o[10.0].nnz, b, b)))
    O.multiply_truncate(1.0, O.Matrix(o[8.0], b, host[0]), O.Matrix(o[6.0], b, host[1]), 0.0, ref)
    A.blocks[A.blocks.shape[0] // 2, 0, b - 1] = float("inf")
    A2 = bsm.Matrix(A.pattern, torch.tensor(host[0], device=ctx.device))
    for prec in (bsm.F64, bsm.F32):
        got = {}
        for variant, tmode in ((0, 1), (-1, 0), (-1, 2)):
            ctx.set_product_variant(variant)
            ctx.set_transposed_plans(tmode)
            print("other b", b, prec, variant, tmode, flush=True)
            C, D = bsm.Matrix(g[10.0]), bsm.Matrix(g[10.0])
            bsm.multiply_truncate_prec(prec, 1.0, A2, B, 0.0, C)
            bsm.multiply_truncate_prec(prec, 1.0, A, B, 0.0, D)
            got[(variant, tmode)] = (C.blocks.cpu().numpy(), D.blocks.cpu().numpy())
        if prec == bsm.F64:
            assert np.abs(got[(0, 1)][0] - ref.blocks).max() <= 1e-12 * np.abs(ref.blocks).max()
        assert not np.isfinite(got[(0, 1)][1]).all()
        for key in ((-1, 0), (-1, 2)):
            assert np.array_equal(got[key][0], got[(0, 1)][0]), key
            if key == (-1, 0):   # the direct plan has the scalar kernel's operand order
                assert np.array_equal(got[key][1], got[(0, 1)][1], equal_nan=True), key
