"""Ring tiles of every height, on systems whose atom count is no multiple of a row group: the last
group's missing rows, direct and transposed, single and paired.

A product of few tiles takes 2 rows and one of 1600 tiles (of 8 rows) or more 8 or 4, so the 637 and
997 atoms here reach the tall tiles of the block sizes that have no setting for them, and the paired
tiles of 8 rows.  All kernels sum the same terms in the same order: results equal the scalar-operand
kernel's (variant 0) bit for bit, and that one is held to the oracle at 1e-12 of its scale
(sums of a few hundred terms of order one: rounding below 1e-13).
"""
import numpy as np
import pytest
import torch

import oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bsm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm


def lattice(cells, drop):
    a = 5.43
    base = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0], [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]]) * (a / 4)
    at = np.stack(np.meshgrid(*[np.arange(m) * a for m in cells], indexing="ij"), -1).reshape(-1, 1, 3)
    pos = (at + base).reshape(-1, 3)
    pos = pos + np.random.default_rng(5).normal(0, 0.1, pos.shape)
    return pos[:len(pos) - drop], [a * m for m in cells]


def draw(bsm, P, seed):
    g = torch.Generator(device=P.ctx.device)
    g.manual_seed(seed)
    return bsm.Matrix(P, 2.0 * torch.rand((P.nnzb, P.b, P.b), dtype=torch.float64, device=P.ctx.device, generator=g) - 1.0)


def rows_of_last_launch(ctx, products=1):
    rows = {s["rows"] for s in ctx.product_stats() if s["products"] == products}
    ctx.set_profiling(True)   # clears the records
    return rows


@pytest.mark.parametrize("cells,drop,tall", [((2, 2, 3), 3, False), ((4, 4, 5), 3, True)])
@pytest.mark.parametrize("b", [5, 6, 7, 8, 10, 11, 12, 13, 14, 15, 16])
def test_other_block_sizes(bsm, b, cells, drop, tall):
    """Also with an infinite element in A and one in B, which reach the blocks of their own triples
    and no others, in either order of the operands."""
    ctx = bsm.Context(0)
    pos, box = lattice(cells, drop)
    P = {r: bsm.Pattern(ctx, pos, box, r, b) for r in (8.0, 6.0, 10.0)}
    A, B, C0 = draw(bsm, P[8.0], 1), draw(bsm, P[6.0], 2), draw(bsm, P[10.0], 3)
    infA, infB = bsm.Matrix(A.pattern, A.blocks.clone()), bsm.Matrix(B.pattern, B.blocks.clone())
    infA.blocks[A.blocks.shape[0] // 2, 0, b - 1] = float("inf")
    infB.blocks[B.blocks.shape[0] // 2, b - 1, 0] = float("inf")
    ctx.set_profiling(True)
    for prec in (bsm.F64, bsm.F32):
        want = None
        for variant, tmode in ((0, 1), (-1, 0), (-1, 2)):
            ctx.set_product_variant(variant)
            ctx.set_transposed_plans(tmode)
            print("other b", b, len(pos), prec, variant, tmode, flush=True)
            got = []
            for x, y, alpha, beta in ((A, B, 1.0, 0.0), (A, B, -0.7, 0.3), (infA, B, 1.0, 0.0), (A, infB, 1.0, 0.0)):
                C = bsm.Matrix(P[10.0], C0.blocks.clone())
                bsm.multiply_truncate_prec(prec, alpha, x, y, beta, C)
                got.append(C.blocks)
            rows = rows_of_last_launch(ctx)
            if variant == 0:
                want = got
                assert all(not bool(torch.isfinite(v).all()) for v in got[2:])
                continue
            assert rows == {(8 if b <= 8 else 4) if tall else 2}
            for k, (v, w) in enumerate(zip(got, want)):
                same = (v == w) | (torch.isnan(v) & torch.isnan(w))
                assert bool(same.all()), (prec, tmode, k)
    ctx.close()


@pytest.mark.parametrize("b,cells,drop", [(4, (5, 5, 5), 3), (9, (5, 5, 5), 3), (4, (2, 2, 3), 1), (9, (2, 2, 3), 1)])
def test_pairs(bsm, b, cells, drop):
    ctx = bsm.Context(0)
    pos, box = lattice(cells, drop)
    P = {r: bsm.Pattern(ctx, pos, box, r, b) for r in (8.0, 6.0, 10.0)}
    A, A2, B, B2 = draw(bsm, P[8.0], 1), draw(bsm, P[8.0], 2), draw(bsm, P[6.0], 3), draw(bsm, P[6.0], 4)
    C0, D0 = draw(bsm, P[10.0], 5), draw(bsm, P[10.0], 6)
    plan_rows = 4 if len(pos) > 500 else 2
    for alpha, beta in ((1.0, 0.0), (-0.7, 0.3)):
        def single(x, y, c0):
            C = bsm.Matrix(P[10.0], c0.blocks.clone())
            bsm.multiply_truncate(alpha, x, y, beta, C)
            return C.blocks
        ctx.set_product_variant(0)
        want = single(A, B, C0), single(A2, B, D0), single(A, B2, D0)
        ctx.set_product_variant(-1)
        assert torch.equal(single(A, B, C0), want[0])
        for name, call, w in (("pair", lambda C, D: bsm.multiply_truncate_pair(alpha, A, A2, B, beta, C, D), want[1]),
                              ("pair_a", lambda C, D: bsm.multiply_truncate_pair_a(alpha, A, B, B2, beta, C, D), want[2])):
            print("pairs", b, len(pos), alpha, name, flush=True)
            C, D = bsm.Matrix(P[10.0], C0.blocks.clone()), bsm.Matrix(P[10.0], D0.blocks.clone())
            ctx.set_profiling(True)
            call(C, D)
            assert rows_of_last_launch(ctx, 2) == {plan_rows}
            assert torch.equal(C.blocks, want[0]) and torch.equal(D.blocks, w), name
    ctx.close()


@pytest.mark.parametrize("drop", [1, 3, 5, 7])
@pytest.mark.parametrize("b", [4, 9, 13])
def test_ragged_row_groups_match_the_oracle(bsm, b, drop):
    ctx = bsm.Context(0)
    pos, box = lattice((2, 2, 2), drop)
    radii = (7.0, 5.0, 8.0)
    P = [bsm.Pattern(ctx, pos, box, r, b) for r in radii]
    o = [O.create_pattern(pos, np.array(box), r) for r in radii]
    ha, hb = (synth.random_blocks(p.nnz, b, 70 + k) for k, p in enumerate(o[:2]))
    ref = O.Matrix(o[2], b, np.zeros((o[2].nnz, b, b)))
    O.multiply_truncate(1.0, O.Matrix(o[0], b, ha), O.Matrix(o[1], b, hb), 0.0, ref)
    A, B = bsm.Matrix(P[0], torch.tensor(ha, device=ctx.device)), bsm.Matrix(P[1], torch.tensor(hb, device=ctx.device))
    first = None
    for variant, rows, tmode in ((0, 0, 0), (-1, 0, 0), (-1, 0, 2)) + (
            () if b == 13 else tuple((-1, r, t) for r in (2, 4, 8) for t in (0, 2))):
        ctx.set_product_variant(variant)
        ctx.set_rows_per_wave(rows)
        ctx.set_transposed_plans(tmode)
        print("ragged", b, len(pos), variant, rows, tmode, flush=True)
        C = bsm.Matrix(P[2])
        bsm.multiply_truncate(1.0, A, B, 0.0, C)
        if first is None:
            first = C.blocks
            assert np.abs(first.cpu().numpy() - ref.blocks).max() <= 1e-12 * np.abs(ref.blocks).max()
        assert torch.equal(C.blocks, first), (variant, rows, tmode)
    ctx.close()
