"""Products on both sides of the lines between tiles of near columns and runs of row sets (a pattern
0.35 full with up to 4 rows a tile of b = 9, else 0.7 or 0.8), and a row group of more columns than the near-column
order holds in LDS (2048: it keeps the row sets).  Every choice sums the same terms in the same
order: results equal those of tiles in ascending columns, bit for bit, and of the scalar-operand
kernel (variant 0).
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm


def check(bsm, n, side, cutoff, b, rows, fill=None):
    ctx = bsm.Context(0)
    g = torch.Generator(device=ctx.device)
    g.manual_seed(n)
    pos = torch.rand((n, 3), dtype=torch.float64, device=ctx.device, generator=g) * side
    P = bsm.Pattern(ctx, pos, (side,) * 3, cutoff, b)
    if fill is not None:
        assert fill[0] < P.nnzb / n ** 2 < fill[1], P.nnzb / n ** 2
    A, B = (bsm.Matrix(P, torch.randn((P.nnzb, b, b), dtype=torch.float64, device=ctx.device, generator=g))
            for _ in range(2))
    out = []
    for variant, order in ((-1, 1), (-1, 0), (0, 1)):
        ctx.set_product_variant(variant)
        ctx.set_column_order(order)
        ctx.set_rows_per_wave(rows)
        print("columns", n, cutoff, b, rows, P.nnzb, variant, order, flush=True)
        C = bsm.Matrix(P)
        bsm.multiply_truncate(1.0, A, B, 0.0, C)
        out.append(C.blocks)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    P.close()
    ctx.close()


# 203 atoms: the last row group has 3
@pytest.mark.parametrize("rows,cutoff,fill", [(2, 8.6, (0.3, 0.35)), (2, 9.0, (0.35, 0.4)), (4, 8.6, (0.3, 0.35)),
                                              (4, 9.0, (0.35, 0.4)), (8, 10.8, (0.6, 0.7)), (8, 11.6, (0.7, 0.8))])
@pytest.mark.parametrize("b", [4, 9, 7])
def test_both_sides_of_the_lines(bsm, b, rows, cutoff, fill):
    check(bsm, 203, 20.0, cutoff, b, rows if b != 7 else 0, fill)


def test_more_columns_than_lds_holds(bsm):
    check(bsm, 2300, 30.0, 12.5, 4, 8, (0.2, 0.35))
