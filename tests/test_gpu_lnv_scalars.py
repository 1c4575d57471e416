"""LNV steps whose scalars stay on the device: block sizes without kernels of their own, the
first steps (no previous direction), and steps that must leave L as it was.

Tolerances: E, N and mu within 1e-10 of the FP64 oracle, relative (traces of some 1e6 terms of
both signs, summed in another order: 1e3 roundings of 1e-16 of sums up to 1e3 times their
result); a refused step leaves L's bits.
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


@pytest.fixture(scope="module")
def ctx(bsm):
    return bsm.Context(0)


def setup(bsm, ctx, b, mode=0, mu=0.0):
    s = synth.make_system("sc", (2, 2, 2), b, synth.SMALL_CUTOFFS, 77)
    pos = torch.tensor(s.positions, dtype=torch.float64, device=ctx.device)
    oP = {k: O.create_pattern(s.positions, s.box, s.cutoffs[k]) for k in ("S", "Z", "L")}
    oS = O.from_blocks(oP["S"], b, s.S.rows, s.S.cols, s.S.blocks)
    oH = O.from_blocks(oP["S"], b, s.H.rows, s.H.cols, s.H.blocks)
    P = {k: bsm.Pattern(ctx, pos, s.box, s.cutoffs[k], b) for k in ("S", "Z", "L")}
    S, H = (bsm.Matrix(P["S"], torch.tensor(m.blocks, device=ctx.device)) for m in (oS, oH))
    Z, L = bsm.Matrix(P["Z"]), bsm.Matrix(P["L"])
    bsm.hotelling_inverse(S, Z, max_iter=10, tol=0.0)
    oZ = O.hotelling_inverse(oS, oP["Z"], max_iter=10, tol=0.0).Z
    return s, S, H, Z, L, oS, oH, oZ, oP


@pytest.mark.parametrize("b,mode,mu", [(4, 1, 0.1), (5, 0, 0.0), (9, 0, 0.0), (13, 0, 0.0)])
def test_first_steps_match_the_oracle(bsm, ctx, b, mode, mu):
    print("lnv scalars b", b, mode, flush=True)
    s, S, H, Z, L, oS, oH, oZ, oP = setup(bsm, ctx, b)
    g = bsm.LNV(S, H, Z, L, s.n_electrons, mode=mode, mu=mu)
    st = O.lnv_init(oS, oH, oZ, oP["L"], s.n_electrons, mode=mode, mu=mu)
    for it in range(4):
        rg, ro = g.step(), O.lnv_step(st)
        assert rg.status == ro.status == 0
        assert abs(rg.E - ro.E) <= 1e-10 * abs(ro.E), (it, rg.E, ro.E)
        assert abs(rg.N - ro.N) <= 1e-10 * abs(ro.N)
        assert abs(rg.mu - ro.mu) <= 1e-10 * max(1.0, abs(ro.mu))
        assert abs(rg.beta - ro.beta) <= 1e-8 * max(1.0, abs(ro.beta))
    g.close()


def test_refused_steps_leave_L(bsm, ctx):
    s, S, H, Z, L, *_ = setup(bsm, ctx, 4)
    L = bsm.Matrix(L.pattern, torch.zeros_like(L.blocks))
    bsm.mask_copy(Z, L)
    L.blocks.mul_(2.0)
    before = L.blocks.clone()
    g = bsm.LNV(S, H, Z, L, s.n_electrons, mode=1, mu=-10.0, init_from_z=False)
    print("lnv runaway", flush=True)
    assert g.step().status == bsm.ERUNAWAY
    assert torch.equal(L.blocks, before)
    g.close()
    bad = H.blocks.clone()
    bad[0, 0, 0] = float("nan")
    print("lnv not finite", flush=True)
    g = bsm.LNV(S, bsm.Matrix(H.pattern, bad), Z, L, s.n_electrons, init_from_z=False)
    r = g.step()
    assert r.status == bsm.ENONFINITE and np.isnan(r.Omega)
    assert torch.equal(L.blocks, before)
    g.close()
