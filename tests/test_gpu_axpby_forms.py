"""axpby on both sides of the line between pairs and single elements, even and odd counts, operands
at and off a 16-byte boundary, with and without reading y: each element is one product and one
fused multiply-add, so all forms give the same bits as the small calls, which the oracle checks.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


# full patterns of n atoms: n^2 b^2 elements, odd where both are odd, on either side of 25 million
@pytest.mark.parametrize("b,n,cutoff", [(3, 5, 100.0), (16, 312, 100.0), (16, 313, 100.0), (15, 333, 100.0), (15, 335, 100.0)])
def test_forms_agree(b, n, cutoff):
    import paper_2205_08941_amd as bsm
    ctx = bsm.Context(0)
    g = torch.Generator(device=ctx.device)
    g.manual_seed(n)
    pos = torch.rand((n, 3), dtype=torch.float64, device=ctx.device, generator=g) * 30.0
    P = bsm.Pattern(ctx, pos, (30.0, 30.0, 30.0), cutoff, b)
    count = P.nnzb * b * b
    print("axpby", b, n, count, flush=True)
    x, y = (torch.randn(count + 1, dtype=torch.float64, device=ctx.device, generator=g) for _ in range(2))
    for beta in (-0.4, 0.0):
        got = []
        for off in (0, 1):
            bx, by = (torch.empty(count + 1, dtype=torch.float64, device=ctx.device) for _ in range(2))
            bx[off:off + count] = x[:count]
            by[off:off + count] = y[:count]
            shape = (P.nnzb, b, b)
            bsm.axpby(0.3, bsm.Matrix(P, bx[off:off + count].view(shape)), beta,
                      bsm.Matrix(P, by[off:off + count].view(shape)))
            got.append(by[off:off + count].clone())
        assert torch.equal(got[0], got[1])
        # 64 bits: one rounding of the product, one of the sum
        want = 0.3 * x[:count] + beta * y[:count]
        scale = (0.3 * x[:count]).abs() + (beta * y[:count]).abs()
        assert bool(((got[0] - want).abs() <= 2.0 ** -52 * scale).all())
    ctx.close()
