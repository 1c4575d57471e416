"""The product planner's device code on the CPU with windows of a few atoms.

The planner holds its rows as bit masks over windows of atoms (k_tile_entries,
k_group_union, k_group_tiles).  Here the window constants are cut down so that a
216-atom cell takes several windows, the last one partial, and every check of
tests/test_planner_host.py runs again: what one window schedules, many must.
"""
import os
import subprocess

import numpy as np
import pytest

import oracle as O
import synth
from test_planner_host import CASES, ROOT, SHIM


@pytest.fixture(scope="module")
def patterns(tmp_path_factory):
    d = tmp_path_factory.mktemp("windows")
    s = synth.make_system("d3", (3, 3, 3), 4, synth.SMALL_CUTOFFS, 6, displacement_sigma=0.1)
    out = {}
    for r in (4.0, 5.0, 7.0):
        P = O.create_pattern(s.positions, s.box, r)
        fn = d / f"p{r}.bin"
        with open(fn, "wb") as f:
            np.array([P.natoms, P.nnz], np.int32).tofile(f)
            P.rowptr.astype(np.int32).tofile(f)
            P.cols.astype(np.int32).tofile(f)
        out[r] = (P, fn)
    return d, out


@pytest.mark.parametrize("words,window", [(1, 64), (2, 50), (6, 1), (7, 216)])
def test_planner_over_many_windows(patterns, words, window):
    d, pats = patterns
    src = open(os.path.join(ROOT, "paper_2205_08941_amd", "csrc", "product.hip")).read()
    a = src.index("// ---------------------------------------------------------------- planner")
    b = src.index("__global__ __launch_bounds__(1024) void k_scan64")
    part = src[a:b]
    for name, value in (("kUnionWords", words), ("kEntryWindow", window)):
        head = part.index(f"constexpr int {name} = ")
        part = part[:head] + f"constexpr int {name} = {value};" + part[part.index(";", head) + 1:]
    cpp, exe = d / f"p{words}_{window}.cpp", d / f"p{words}_{window}"
    cpp.write_text(SHIM + part + open(os.path.join(ROOT, "tests", "host", "planner_main.cpp")).read())
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", str(exe), str(cpp)], check=True)
    for G, JT, W, order, tr in ((8, 7, 1, 1, 0), (16, 7, 1, 1, 0), (4, 16, 2, 1, 0), (8, 16, 1, 0, 1)):
        for ra, rb, rc in CASES:
            (PA, fa), (PB, fb), (PC, fc) = pats[ra], pats[rb], pats[rc]
            r = subprocess.run([str(exe), str(fa), str(fb), str(fc), str(G), str(JT), str(W), str(order), str(tr), "2"],
                               capture_output=True, text=True, timeout=120)
            seen, bad = (int(v) for v in r.stdout.split())
            assert r.returncode == 0 and bad == 0, (G, JT, W, order, tr, ra, rb, rc, r.stdout)
            assert seen == int(O.count_triples(PA, PB, PC).sum()), (ra, rb, rc)
