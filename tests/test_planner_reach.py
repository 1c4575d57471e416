"""The product planner's work on a long system (its device code on the CPU, no GPU needed).

A chain of 40000 atoms, each with the three next on either side: a tile reaches some 20 of
them.  Planning it must cost what it reaches.  The planner's barriers are counted (plan_sync, a few per window of
1024 atoms): one or two windows a tile, not the 40 of the whole chain; and every check of
tests/host/planner_main.cpp holds.
"""
import os
import re
import subprocess

import numpy as np
import pytest

import oracle as O
import synth
from test_planner_host import CASES, ROOT, SHIM

N, REACH = 40000, 3


@pytest.mark.parametrize("ring", [False, True])
def test_planner_skips_windows_no_tile_reaches(tmp_path, ring):
    """ring: the chain closed, so that the rows at its ends reach the first and the last window."""
    src = open(os.path.join(ROOT, "paper_2205_08941_amd", "csrc", "product.hip")).read()
    a = src.index("// ---------------------------------------------------------------- planner")
    b = src.index("__global__ __launch_bounds__(1024) void k_scan64")
    part = src[a:b]
    count = ("static struct Syncs { long n = 0; ~Syncs() { std::fprintf(stderr, \"%ld\\n\", n); } } syncs;\n"
             "inline void plan_sync() { ++syncs.n; }")
    assert part.count("inline void plan_sync() {}") == 1
    part = part.replace("inline void plan_sync() {}", count)
    cpp, exe = tmp_path / "reach.cpp", tmp_path / "reach"
    cpp.write_text("#include <cstdio>\n" + SHIM + part +
                   open(os.path.join(ROOT, "tests", "host", "planner_main.cpp")).read())
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", str(exe), str(cpp)], check=True)
    off = np.arange(-REACH, REACH + 1)
    cols = np.arange(N)[:, None] + off
    keep = np.ones(cols.shape, bool) if ring else (cols >= 0) & (cols < N)
    rows = [np.sort(c[k] % N) for c, k in zip(cols, keep)]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    with open(tmp_path / "p.bin", "wb") as f:
        np.array([N, rp[-1]], np.int32).tofile(f)
        rp.astype(np.int32).tofile(f)
        np.concatenate(rows).astype(np.int32).tofile(f)
    p = str(tmp_path / "p.bin")
    r = subprocess.run([str(exe), p, p, p, "8", "7", "1", "1", "0", "1"], capture_output=True, text=True, timeout=120)
    seen, bad = (int(v) for v in r.stdout.split())
    assert r.returncode == 0 and bad == 0, r.stdout
    # triples (i, k, j): pairs of steps of at most REACH that add up to at most REACH
    per = sum(1 for x in off for y in off if abs(x + y) <= REACH)
    assert seen == per * N if ring else 0.999 * per * N < seen < per * N
    groups = N // 8
    tiles = 2 * groups   # 14 columns, 7 a tile
    # a group: fewer than 20 barriers for its tiles' columns and their sort; a tile: counted and
    # written, each 1 before its windows and at most 5 in one, one window and sometimes two
    assert int(re.search(r"(\d+)", r.stderr).group(1)) <= 20 * groups + 2 * tiles * (1 + 5 * 1.5)


@pytest.mark.parametrize("words,window", [(1, 64), (2, 50), (6, 1), (7, 216)])
def test_planner_over_many_windows_in_one_chunk(tmp_path, words, window):
    """Windows of a few atoms, each tile walking all its k as on the GPU (one chunk)."""
    src = open(os.path.join(ROOT, "paper_2205_08941_amd", "csrc", "product.hip")).read()
    a = src.index("// ---------------------------------------------------------------- planner")
    b = src.index("__global__ __launch_bounds__(1024) void k_scan64")
    part = src[a:b]
    for name, value in (("kUnionWords", words), ("kEntryWindow", window)):
        head = part.index(f"constexpr int {name} = ")
        part = part[:head] + f"constexpr int {name} = {value};" + part[part.index(";", head) + 1:]
    cpp, exe = tmp_path / "w.cpp", tmp_path / "w"
    cpp.write_text(SHIM + part + open(os.path.join(ROOT, "tests", "host", "planner_main.cpp")).read())
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", str(exe), str(cpp)], check=True)
    s = synth.make_system("d3", (3, 3, 3), 4, synth.SMALL_CUTOFFS, 6, displacement_sigma=0.1)
    files, pats = {}, {}
    for r in (4.0, 5.0, 7.0):
        pats[r] = P = O.create_pattern(s.positions, s.box, r)
        files[r] = str(tmp_path / f"p{r}.bin")
        with open(files[r], "wb") as f:
            np.array([P.natoms, P.nnz], np.int32).tofile(f)
            P.rowptr.astype(np.int32).tofile(f)
            P.cols.astype(np.int32).tofile(f)
    for G, JT, W, order, tr in ((8, 7, 1, 1, 0), (2, 16, 1, 1, 1), (4, 16, 2, 1, 0), (8, 16, 1, 0, 1)):
        for ra, rb, rc in CASES:
            r = subprocess.run([str(exe), files[ra], files[rb], files[rc], str(G), str(JT), str(W), str(order),
                                str(tr), "1"], capture_output=True, text=True, timeout=120)
            seen, bad = (int(v) for v in r.stdout.split())
            assert r.returncode == 0 and bad == 0, (G, JT, W, order, tr, ra, rb, rc, r.stdout)
            assert seen == int(O.count_triples(pats[ra], pats[rb], pats[rc]).sum()), (ra, rb, rc)
