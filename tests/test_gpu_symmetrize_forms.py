"""symmetrize on both sides of the line between one and four elements a thread (2^21 elements; always
one for b <= 3): each pair is half the sum of its two elements, exactly.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n", [(1, 7), (3, 483), (3, 484), (4, 362), (4, 363), (9, 160), (9, 161), (13, 111), (13, 112)])
def test_full_matrices(b, n):
    import paper_2205_08941_amd as bsm
    ctx = bsm.Context(0)
    g = torch.Generator(device=ctx.device)
    g.manual_seed(n)
    pos = torch.rand((n, 3), dtype=torch.float64, device=ctx.device, generator=g) * 20.0
    P = bsm.Pattern(ctx, pos, (20.0, 20.0, 20.0), 100.0, b)   # full: slot i n + j
    print("symmetrize", b, n, P.nnzb * b * b, flush=True)
    M = bsm.Matrix(P, torch.randn((P.nnzb, b, b), dtype=torch.float64, device=ctx.device, generator=g))
    full = M.blocks.view(n, n, b, b).clone()
    bsm.symmetrize(M)
    assert torch.equal(M.blocks.view(n, n, b, b), 0.5 * (full + full.permute(1, 0, 3, 2)))
    ctx.close()
