"""GPU tests of the rules that choose a Krylov step's kernels, read back from
the library: which matrices and blocks take which product and which instances,
at the sizes where the rules change."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu

NUG = 2e-2


@pytest.fixture(scope="module")
def L():
    from paper_2606_07004_amd import liblogdet
    liblogdet.lib()  # fails loudly when the HIP library is missing
    return liblogdet


@pytest.fixture(scope="module")
def ctx(L):
    c = L.Context(0)
    yield c
    c.close()


def _csr(m):
    m = sp.csr_matrix(m)
    m.sort_indices()
    return W.Csr(m.shape[0], m.indptr.astype(np.int32), m.indices.astype(np.int32),
                 m.data.astype(np.float64))


def _stripes(n, strides):
    """Constant diagonals at the given offsets, diagonally dominant."""
    strides = [s for s in strides if s < n]
    offs = [0] + strides + [-s for s in strides]
    return _csr(sp.diags([2.0 * len(strides) + 0.5] + [-1.0] * (2 * len(strides)), offs,
                         shape=(n, n)))


def _paths(L, ctx, a, npr, prec="mixed", vt="fp32", k=2, lo=0.0, pin=None):
    h = ctx.matrix(a, vt={"fp64": L.LD_VT_FP64, "fp32": L.LD_VT_FP32, "bf16": L.LD_VT_BF16}[vt],
                   lo_hint=lo)
    try:
        p = L.make_params(npr, max(1, npr // 3), 8, k, 3, precision={
            "fp64": L.LD_PREC_FP64, "mixed": L.LD_PREC_MIXED, "half": L.LD_PREC_HALF}[prec])
        if pin is not None:
            L.ld_tune_set(h, p, *pin)
        print(f"\n[case] step paths n={a.n} probes {npr} {prec} values {vt} window {k} pin {pin}",
              flush=True)
        return L.ld_debug_step_paths(h, p)
    finally:
        ctx.release(h)


def test_products(L, ctx):
    # a covariance keeps tiles; blocks under 16 columns take its row groups; a
    # Laplacian keeps neither; FP16 vectors and BF16 values take the CSR rows
    cov, lap = W.wendland(3001, 48.0, NUG, seed=1), W.lap3d(12, 0.1)
    for prec, vt in (("mixed", "fp32"), ("fp64", "fp64"), ("mixed", "fp64")):
        got = _paths(L, ctx, cov, 30, prec, vt, lo=NUG)
        assert got["product"] == 2 and got["tiles"] == 47 and 200 < got["tile_union"] <= 600
        assert _paths(L, ctx, lap, 30, prec, vt)["product"] == 0
    assert _paths(L, ctx, cov, 13, lo=NUG)["product"] == 2
    assert _paths(L, ctx, cov, 12, lo=NUG)["product"] == 0
    assert _paths(L, ctx, cov, 12, lo=NUG, pin=(3, 1, 3, 1, 1, 0, 0, 1, 1))["product"] == 1
    assert _paths(L, ctx, cov, 30, "half", lo=0.3)["product"] == 0
    got = _paths(L, ctx, cov, 30, vt="bf16", lo=NUG)
    assert got["product"] == got["tiles"] == got["tile_union"] == 0
    # a tile's union too large for LDS: row groups
    wide = W.wendland_grid(40, 50, 24.0, nugget=0.5)
    got = _paths(L, ctx, wide, 30, lo=0.5)
    assert got["product"] == 1 and got["tiles"] == 0


# rows of 8 chunks (30 FP32 probes): 32 rows a chunk of rows; 4, 2 and 1 chunks
# of a row: 64, 128 and 256
@pytest.mark.parametrize("n,npr,prec,vt,k,latency", [
    (32 * 3072, 30, "mixed", "fp32", 2, 1), (32 * 3072 + 1, 30, "mixed", "fp32", 2, 0),
    (32 * 3072, 30, "mixed", "fp64", 2, 1), (16 * 3072, 30, "fp64", "fp64", 10, 1),
    (20000, 16, "mixed", "fp32", 2, 1), (20000, 8, "mixed", "fp32", 2, 0),
    (20000, 4, "mixed", "fp64", 2, 0), (20000, 4, "fp64", "fp64", 2, 0),
    (20000, 8, "fp64", "fp64", 2, 1), (20000, 64, "half", "fp32", 2, 0),
])
def test_latency_instance(L, ctx, n, npr, prec, vt, k, latency):
    got = _paths(L, ctx, _stripes(n, (1, 37)), npr, prec, vt, k)
    assert got["product"] == 0 and got["latency"] == latency


# the update that reads a row ahead: rows of less than a line (7 chunks and
# fewer) up to 320 chunks of rows, FP16 ones past 1024 again; wider rows up to 24
# (12) rounds of 2048 chunks
@pytest.mark.parametrize("n,npr,prec,k,ahead", [
    (256 * 320, 4, "mixed", 2, 1), (256 * 320 + 1, 4, "mixed", 2, 0),
    (32 * 320, 28, "mixed", 2, 1), (32 * 320 + 1, 28, "mixed", 2, 0),
    (32 * 320 + 1, 30, "mixed", 2, 1), (256 * 320 + 1, 2, "fp64", 2, 0),
    (128 * 320, 4, "fp64", 3, 1), (128 * 320 + 1, 4, "fp64", 3, 0), (64 * 320 + 1, 8, "fp64", 3, 1),
    (64 * 320 + 1, 30, "half", 2, 0), (64 * 1024 + 1, 30, "half", 2, 1),
    (16 * 24 * 2048, 64, "mixed", 2, 1), (16 * 24 * 2048 + 1, 64, "mixed", 2, 0),
    (16 * 12 * 2048, 30, "fp64", 4, 1), (16 * 12 * 2048 + 1, 30, "fp64", 4, 0),
    (16 * 12 * 2048 + 1, 30, "fp64", 2, 1), (3000, 30, "mixed", 6, 0),
])
def test_update_ahead(L, ctx, n, npr, prec, k, ahead):
    assert _paths(L, ctx, _stripes(n, (1,)), npr, prec, k=k)["update_ahead"] == ahead
