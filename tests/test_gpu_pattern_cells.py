"""Patterns at the edges of the cell walk: 1, 2, 3 and more cells along each axis (the
walk along z is one run of cells or two where it wraps), runs of fewer and more atoms
than a wavefront has lanes, a single atom, atoms on cell faces and outside the box.

Columns and row pointers are whole numbers: they equal the oracle's.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_08941_amd as bsm
    return bsm.Context(0)


@pytest.mark.parametrize("n,box,cutoff", [
    (1, (5.0, 5.0, 5.0), 3.0),
    (130, (10.0, 10.0, 10.0), 12.0),      # one cell
    (300, (10.0, 10.0, 7.9), 4.0),        # 2, 2, 1 cells
    (700, (10.0, 8.0, 10.0), 3.3),        # 3, 2, 3
    (700, (4.0, 5.0, 40.0), 2.0),         # 2, 2, 20
    (900, (9.0, 40.0, 4.0), 3.0),         # 3, 13, 1
    (515, (13.0, 13.0, 13.0), 2.5),       # 5, 5, 5
])
def test_pattern_of_cells(ctx, n, box, cutoff):
    import paper_2205_08941_amd as bsm
    print("pattern of cells", n, box, cutoff, flush=True)
    rng = np.random.default_rng(n)
    box = np.array(box)
    pos = rng.uniform(-0.5, 1.5, (n, 3)) * box
    pos[::7] = np.round(pos[::7] / box * 4) / 4 * box      # cell faces and box faces
    P = bsm.Pattern(ctx, torch.tensor(pos, dtype=torch.float64, device=ctx.device), box, cutoff, 4)
    rp, cols = P.to_host()
    want = O.create_pattern(pos, box, cutoff)
    assert np.array_equal(rp, want.rowptr) and np.array_equal(cols, want.cols)
    P.close()
