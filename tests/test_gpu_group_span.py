"""bsm_ctx_set_group_span: 0 restores the default order, other values out of range stay refused,
and a product's bits do not depend on the launch order."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def test_zero_restores_the_default():
    import paper_2205_08941_amd as bsm
    ctx = bsm.Context(0)
    s = synth.make_system("span", (2, 2, 2), 4, synth.SMALL_CUTOFFS, 3, displacement_sigma=0.1)
    P = bsm.Pattern(ctx, s.positions, s.box, 6.0, 9)
    A = bsm.Matrix(P, torch.tensor(synth.random_blocks(P.nnzb, 9, 5), device=ctx.device))
    out = []
    for span in (None, 7, 0):
        if span is not None:
            ctx.set_group_span(span)
        C = bsm.Matrix(P)
        bsm.multiply_truncate(1.0, A, A, 0.0, C)
        out.append(C.blocks)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
    for span in (-1, 4097):
        with pytest.raises(bsm.BSMError):
            ctx.set_group_span(span)
    ctx.close()
