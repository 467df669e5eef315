"""CPU test of the walk over a CSR row's entries: the lanes of a row take every
entry once, lane l those at l, l + L, ... in order, also in a row that ends at
2^31 - 1, the largest entry count of a matrix.  entry_walk.h is compiled for the
host, with signed overflow wrapping (as it does on the GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAST = 2 ** 31 - 1


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("entrywalk") / "entry_walk_host"
    src = os.path.join(ROOT, "tests", "csrc", "entry_walk_host.cpp")
    inc = os.path.join(ROOT, "paper_2606_07004_amd", "csrc")
    subprocess.run([gxx, "-O1", "-std=c++17", "-fwrapv", "-I" + inc, src, "-o", str(out)],
                   check=True)
    return str(out)


@pytest.mark.parametrize("end", [1000, LAST - 200, LAST])
def test_lanes_take_every_entry_once(exe, end):
    cases = [(end - cnt, end, L) for cnt in (0, 1, 3, 4, 63, 64, 65, 255, 256, 257, 700)
             for L in (2, 4, 16, 64)]
    out = subprocess.run([exe], input="\n".join("%d %d %d" % c for c in cases),
                         capture_output=True, text=True, check=True).stdout
    lines = out.strip().split("\n")
    assert len(lines) == len(cases)
    for (kb, ke, L), ln in zip(cases, lines):
        want = " ".join(" ".join(str(k) for k in list(range(kb + l, ke, L)) + [-1])
                        for l in range(L))
        assert ln.strip() == want, (kb, ke, L)
