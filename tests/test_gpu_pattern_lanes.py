"""Patterns on both sides of the lines between 16 lanes and a wavefront to an atom: runs of cells of
some 40 atoms, and 16384 atoms; counts that fill no workgroup.  Whole numbers: they equal the oracle's.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,box,cutoff", [
    (349, (12.0, 12.0, 12.0), 4.0),       # 3, 3, 3 cells: runs of 38.8 atoms
    (361, (12.0, 12.0, 12.0), 4.0),       # 40.1
    (977, (8.0, 8.0, 60.0), 4.0),         # 2, 2, 15: 48.9
    (16381, (40.0, 40.0, 40.0), 10.0),    # 4, 4, 4: 768
    (16385, (40.0, 40.0, 40.0), 10.0),
])
def test_both_widths(n, box, cutoff):
    import paper_2205_08941_amd as bsm
    ctx = bsm.Context(0)
    print("pattern lanes", n, box, cutoff, flush=True)
    pos = np.random.default_rng(n).uniform(0.0, 1.0, (n, 3)) * box
    P = bsm.Pattern(ctx, torch.tensor(pos, device=ctx.device), box, cutoff, 1)
    rp, cols = P.to_host()
    want = O.create_pattern(pos, np.array(box), cutoff)
    assert np.array_equal(rp, want.rowptr) and np.array_equal(cols, want.cols)
    ctx.close()
