"""BF16 products of two matrices on one pattern (b = 9) run on the matrix cores over the tiles
of their class's plan.  Their bits must come from the operands alone, whatever kernel variant is
set and whatever ran before, and the class keeps one plan for every precision: no second one is
built, or not, by how much device memory happens to be free.

512 displaced atoms, 8 A: a tile lists some of the atoms only, so that the tiles of near columns
that FP64 products take list others than row-set runs would.
"""
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


def operands(bsm, ctx):
    s = synth.make_system("bf", (4, 4, 4), 4, synth.SMALL_CUTOFFS, 13, displacement_sigma=0.1)
    P = bsm.Pattern(ctx, s.positions, s.box, 8.0, 9)
    A, B = (bsm.Matrix(P, torch.tensor(synth.random_blocks(P.nnzb, 9, k), device=ctx.device)) for k in (61, 62))
    return P, A, B


def product(bsm, P, A, B, prec):
    C = bsm.Matrix(P)
    bsm.multiply_truncate_prec(prec, 1.0, A, B, 0.0, C)
    return C.blocks.clone()


@pytest.mark.parametrize("rows", [4, 8])
def test_bits_do_not_depend_on_variant_or_history(bsm, rows):
    ctx = bsm.Context(0)
    P, A, B = operands(bsm, ctx)
    ctx.set_rows_per_wave(rows)
    ref = product(bsm, P, A, B, bsm.BF16)
    f64 = product(bsm, P, A, B, bsm.F64)   # after BF16
    for variant in (3, 4, 5, 6):
        ctx.set_product_variant(variant)
        print("bf16 variant", variant, rows, flush=True)
        assert torch.equal(product(bsm, P, A, B, bsm.BF16), ref), variant
    ctx.set_product_variant(-1)
    assert torch.equal(product(bsm, P, A, B, bsm.F64), f64)   # before BF16
    assert torch.equal(product(bsm, P, A, B, bsm.BF16), ref)
    ctx.close()


@pytest.mark.parametrize("first", [0, 2])
def test_one_plan_serves_every_precision(bsm, first):
    """What a second precision of the class allocates: the packed operands, 288 bytes a block
    each (BF16 after FP64), or nothing."""
    ctx = bsm.Context(0)
    P, A, B = operands(bsm, ctx)
    ctx.set_rows_per_wave(8)
    second = bsm.F64 + bsm.BF16 - first
    held = lambda: sum(t.numel() for t in ctx._keep.values())
    product(bsm, P, A, B, first)
    before = held()
    product(bsm, P, A, B, second)
    assert held() - before == (2 * 288 * P.nnzb if second == bsm.BF16 else 0)
    ctx.close()
