"""CPU test of the product's band walk: whatever the matrix size, the stride,
the rows per chunk and the grid, every chunk of rows goes to exactly one block,
and chunks a stride apart to blocks of the same XCD (block % 8) but for the
edges of the bands.  band_walk.h is compiled for the host."""
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
    out = tmp_path_factory.mktemp("bandwalk") / "band_walk_host"
    src = os.path.join(ROOT, "tests", "csrc", "band_walk_host.cpp")
    inc = os.path.join(ROOT, "paper_2606_07004_amd", "csrc")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I" + inc, src, "-o", str(out)], check=True)
    return str(out)


def test_band_walk_partitions_the_chunks(exe):
    cases = [(n, stride, rpc, nbk)
             for n in (1, 2049, 40000, 227000)
             for stride in (2048, 2049, 3721, 16384, 65000, 300000)
             for rpc in (4, 12, 20, 32) if stride >= 64 * rpc
             for nbk in (8, 16, 1280, 1536)]
    inp = "\n".join("%d %d %d %d" % c for c in cases)
    out = subprocess.run([exe], input=inp, capture_output=True, text=True, check=True).stdout
    lines = out.strip().split("\n")
    assert len(lines) == len(cases)
    for (n, stride, rpc, nbk), ln in zip(cases, lines):
        v = np.array([int(x) for x in ln.split()])[1:]
        nchunk = -(-n // rpc)
        ends = np.flatnonzero(v == -1)
        assert len(ends) == nbk
        block = np.searchsorted(ends, np.arange(len(v)))
        kept = v >= 0
        ch, xcd = v[kept], block[kept] % 8
        assert np.array_equal(np.sort(ch), np.arange(nchunk))
        where = np.empty(nchunk, int)
        where[ch] = xcd
        # the chunk a stride (rounded down) further: at most one chunk off per
        # band edge, plus the drift of a stride that is no multiple of a chunk
        d = stride // rpc
        if nchunk > 2 * d:
            same = np.mean(where[:-d] == where[d:])
            assert same >= 1 - 2.5 * 8 / d
