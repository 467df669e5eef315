"""CPU test of the choice of the row tiles' shape: the sampled tiles' distinct
columns against sets, and the shape with the fewer of them.  tile_sample.h is
compiled for the host."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("tilesample") / "tile_sample_host"
    src = os.path.join(ROOT, "tests", "csrc", "tile_sample_host.cpp")
    inc = os.path.join(ROOT, "paper_2606_07004_amd", "csrc")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I" + inc, src, "-o", str(out)], check=True)
    return str(out)


def _tiles(n, sg):
    """The groups of every tile: consecutive, or 4 groups on each of 4 lines."""
    ng, out, rest = (n + 3) // 4, [], 0
    if sg and ng // (4 * sg):
        for band in range(ng // (4 * sg)):
            for x in range(0, sg, 4):
                out.append([(4 * band + line) * sg + x + i for line in range(4) for i in range(4)
                            if x + i < sg])
        rest = ng // (4 * sg) * 4 * sg
    return out + [list(range(g, min(ng, g + 16))) for g in range(rest, ng, 16)]


def _sample(a, sg):
    tiles = _tiles(a.n, sg)
    ns = min(len(tiles), 8)
    cols = lambda t: np.unique(np.concatenate(
        [a.col_idx[a.row_ptr[4 * g]:a.row_ptr[min(a.n, 4 * g + 4)]] for g in t]))
    return sum(len(cols(tiles[(2 * i + 1) * len(tiles) // (2 * ns)])) for i in range(ns)) / ns


def _line_groups(a):
    """The middle row's next run of columns after the diagonal's: the offset to
    its centre, in groups."""
    r = a.n // 2
    c = a.col_idx[a.row_ptr[r]:a.row_ptr[r + 1]].astype(int)
    runs = [x for x in np.split(c, np.flatnonzero(np.diff(c) != 1) + 1) if x[0] > r]
    return ((runs[0][0] + runs[0][-1]) // 2 - r + 2) // 4 if runs else 0


# grids on lines of 48, 50 and 47 rows, scattered points, less than a tile, one row
@pytest.mark.parametrize("make", [
    lambda: W.wendland_grid(40, 48, 5.0), lambda: W.wendland_grid(33, 50, 3.5),
    lambda: W.wendland_grid(41, 47, 8.0), lambda: W.wendland(3001, 48.0, 1e-2, seed=3),
    lambda: W.wendland(45, 20.0, 1e-2, seed=3), lambda: W.diag_matrix([2.0]),
    lambda: W.lap2d(60, 0.1)])
def test_shape_of_the_smaller_union(exe, make):
    a = make()
    sgs = [0, 12, max(4, _line_groups(a))]
    inp = " ".join(map(str, [a.n, a.nnz, len(sgs)] + sgs + list(a.row_ptr) + list(a.col_idx)))
    out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout.split()
    want = [_sample(a, sg) for sg in sgs]
    assert [float(x) for x in out[2:]] == want
    grid = _line_groups(a) >= 4 and want[2] < want[0]
    assert (int(out[0]), int(out[1])) == ((4, sgs[2]) if grid else (16, 0))
