"""CPU test of the row-tile product's tile shapes: whatever the matrix size and
line stride, the tiles partition the row groups (each group in exactly one
tile), so every row is written once.  row_tiles.h is compiled for the host."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("rowtiles") / "row_tiles_host"
    src = os.path.join(ROOT, "tests", "csrc", "row_tiles_host.cpp")
    inc = os.path.join(ROOT, "paper_2606_07004_amd", "csrc")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I" + inc, src, "-o", str(out)], check=True)
    return str(out)


def test_tiles_partition_the_groups(exe):
    # consecutive groups; bands of 4 lines with whole and ragged tiles per
    # line, partial last bands, lines longer than the matrix
    cases = [(n, sg, gx) for n in (1, 3, 4, 63, 64, 65, 257, 1000, 4001, 20000)
             for sg, gx in ((0, 0), (4, 4), (5, 4), (7, 4), (30, 4), (63, 4), (300, 4), (9, 8),
                            (40, 2), (40, 16), (40, 3))]
    inp = "\n".join("%d %d %d" % c for c in cases)
    out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout
    lines = out.strip().split("\n")
    assert len(lines) == len(cases)
    for (n, sg, gx), ln in zip(cases, lines):
        v = np.array([int(x) for x in ln.split()])
        ng = (n + 3) // 4
        tiles = v[3:].reshape(v[2], 16)
        kept = np.sort(tiles[tiles >= 0])
        assert np.array_equal(kept, np.arange(ng)), (n, sg, gx)
        if v[1]:  # bands: a full tile's groups lie on 16 / gx lines, gx each
            assert (v[0], v[1]) == (gx, sg)
            full = tiles[0]
            if (full >= 0).all():
                want = (np.arange(16 // gx)[:, None] * sg + np.arange(gx)[None, :]).ravel()
                assert np.array_equal(full, want)
