"""How the ring tiles copy b = 4 blocks (and b = 9 past 4 GB): packed (16 bytes a lane) from any 8-byte boundary, through
buffer resources or, for variant 3 and for operands past 4 GB, with 64-bit addresses; a block to a
load only off 8-byte boundaries.  Every form sums the same terms in the same order: results equal
the scalar-operand kernel's (variant 0) bit for bit.
"""
import ctypes

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm


def moved(bsm, M, nbytes):
    """M with its blocks nbytes past an aligned address."""
    n = M.blocks.numel() * 8
    raw = torch.empty(n + 64, dtype=torch.uint8, device=M.blocks.device)
    raw[nbytes:nbytes + n].copy_(M.blocks.reshape(-1).view(torch.uint8))
    out = bsm.Matrix(M.pattern, M.blocks)
    out._raw = raw
    out._c = type(M._c)(M.pattern.handle, bsm.F64, ctypes.c_void_p(raw.data_ptr() + nbytes))
    return out


def operands(bsm, ctx, cells=(2, 2, 3), drop=3, radii=(8.0, 6.0, 10.0)):
    s = synth.make_system("pack", cells, 4, synth.SMALL_CUTOFFS, 23, displacement_sigma=0.1)
    pos = np.asarray(s.positions)[:len(s.positions) - drop]
    P = [bsm.Pattern(ctx, pos, s.box, r, 4) for r in radii]
    M = [bsm.Matrix(p, torch.tensor(synth.random_blocks(p.nnzb, 4, 90 + k), device=ctx.device))
         for k, p in enumerate(P[:2])]
    A2 = bsm.Matrix(P[0], torch.tensor(synth.random_blocks(P[0].nnzb, 4, 95), device=ctx.device))
    B2 = bsm.Matrix(P[1], torch.tensor(synth.random_blocks(P[1].nnzb, 4, 96), device=ctx.device))
    return P, M[0], A2, M[1], B2


def reference(bsm, ctx, P, A, B):
    ctx.set_product_variant(0)
    C = bsm.Matrix(P)
    bsm.multiply_truncate(1.0, A, B, 0.0, C)
    ctx.set_product_variant(-1)
    return C.blocks


@pytest.mark.parametrize("offset", [0, 4, 8])
@pytest.mark.parametrize("variant,rows", [(-1, 2), (-1, 4), (-1, 8), (3, 2), (3, 4), (3, 8), (5, 4), (5, 8)])
def test_copies_of_every_variant(bsm, variant, rows, offset):
    ctx = bsm.Context(0)
    P, A, A2, B, B2 = operands(bsm, ctx)
    ref = reference(bsm, ctx, P[2], A, B)
    mA, mB = moved(bsm, A, offset), moved(bsm, B, offset)
    for tmode in (0, 2):
        ctx.set_product_variant(variant)
        ctx.set_rows_per_wave(rows)
        ctx.set_transposed_plans(tmode)
        print("packed", variant, rows, offset, tmode, flush=True)
        C = bsm.Matrix(P[2])
        bsm.multiply_truncate(1.0, mA, mB, 0.0, C)
        assert torch.equal(C.blocks, ref), tmode
    ctx.close()


@pytest.mark.parametrize("offset", [0, 4, 8])
def test_copies_of_pairs_and_batches(bsm, offset):
    ctx = bsm.Context(0)
    P, A, A2, B, B2 = operands(bsm, ctx)
    want = {k: reference(bsm, ctx, P[2], x, y) for k, x, y in (("AB", A, B), ("A2B", A2, B), ("AB2", A, B2))}
    mA, mA2, mB, mB2 = (moved(bsm, M, offset) for M in (A, A2, B, B2))
    C, D = bsm.Matrix(P[2]), bsm.Matrix(P[2])
    print("packed pairs", offset, flush=True)
    bsm.multiply_truncate_pair(1.0, mA, mA2, mB, 0.0, C, D)
    assert torch.equal(C.blocks, want["AB"]) and torch.equal(D.blocks, want["A2B"])
    bsm.multiply_truncate_pair_a(1.0, mA, mB, mB2, 0.0, C, D)
    assert torch.equal(C.blocks, want["AB"]) and torch.equal(D.blocks, want["AB2"])
    P9 = bsm.Pattern(ctx, synth.make_system("p9", (2, 2, 2), 4, synth.SMALL_CUTOFFS, 3).positions, (10.86,) * 3, 6.0, 9)
    A9 = bsm.Matrix(P9, torch.tensor(synth.random_blocks(P9.nnzb, 9, 99), device=ctx.device))
    want9 = reference(bsm, ctx, P9, A9, A9)
    for mixed in (False, True):   # b = 4 alone, and beside b = 9
        C, D, E = bsm.Matrix(P[2]), bsm.Matrix(P[2]), bsm.Matrix(P9)
        bt = bsm.Batch(ctx, [(mA, mB, C), (mA2, mB, D)] + ([(moved(bsm, A9, offset), A9, E)] if mixed else []))
        for mode in (bsm.BATCH_ONE_LAUNCH, bsm.BATCH_PER_B):
            print("packed batch", offset, mixed, mode, flush=True)
            for M in (C, D, E):
                M.blocks.fill_(float("nan"))
            bt.run(order=bsm.ORDER_BY_PRODUCT, mode=mode)
            assert torch.equal(C.blocks, want["AB"]) and torch.equal(D.blocks, want["A2B"])
            assert not mixed or torch.equal(E.blocks, want9)
        bt.close()
    ctx.close()


@pytest.mark.parametrize("n,b,side", [(5800, 4, 49.0), (2580, 9, 37.0)])
def test_operands_past_4_GB(bsm, n, b, side):
    """A full pattern: 4.3 GB of blocks, past a buffer resource."""
    ctx = bsm.Context(0)
    g = torch.Generator(device=ctx.device)
    g.manual_seed(7)
    pos = torch.rand((n, 3), dtype=torch.float64, device=ctx.device, generator=g) * side
    box = (side,) * 3
    W, N = bsm.Pattern(ctx, pos, box, 100.0, b), bsm.Pattern(ctx, pos, box, 6.0, b)
    assert W.nnzb * b * b * 8 > 0xfffff000
    draw = lambda P: bsm.Matrix(P, torch.randn((P.nnzb, b, b), dtype=torch.float64, device=ctx.device, generator=g))
    A, A2, B, B2 = draw(W), draw(W), draw(N), draw(N)
    want = {k: reference(bsm, ctx, N, x, y) for k, x, y in (("AB", A, B), ("A2B", A2, B), ("AB2", A, B2))}
    C, D = bsm.Matrix(N), bsm.Matrix(N)
    for tmode in (0, 2):
        ctx.set_transposed_plans(tmode)
        print("past 4 GB", b, tmode, flush=True)
        bsm.multiply_truncate(1.0, A, B, 0.0, C)
        assert torch.equal(C.blocks, want["AB"]), tmode
    print("pairs past 4 GB", b, flush=True)
    bsm.multiply_truncate_pair(1.0, A, A2, B, 0.0, C, D)
    assert torch.equal(C.blocks, want["AB"]) and torch.equal(D.blocks, want["A2B"])
    bsm.multiply_truncate_pair_a(1.0, A, B, B2, 0.0, C, D)
    assert torch.equal(C.blocks, want["AB"]) and torch.equal(D.blocks, want["AB2"])
    ctx.close()
    torch.cuda.empty_cache()
