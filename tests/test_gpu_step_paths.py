"""GPU tests of the CSR product's and update's instances: the latency instance
for few chunks of rows per block and the band walk for matrices with a frequent
large stride, each at the sizes where its rule or its remainders change.

Every case is run in the default geometry and in a pinned one that takes the
general path over the same matrix (two chunks per lane; interleaved chunks).
A row's product is the same FMA chain in both, and only the order of the FP64
partial sums of inner products differs (each to about 1e-14 of its size), so
per-probe values agree to 1e-10 with FP64 vectors.  With FP32 (FP16) vectors a
changed last bit of a coefficient can move single entries by one rounding,
2^-24 (2^-11) of the entry, hence 1e-6 (5e-4).
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-6, "half": 5e-4}


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
    import workloads as W
    m = sp.csr_matrix(m)
    m.sort_indices()
    return W.Csr(m.shape[0], m.indptr.astype(np.int32), m.indices.astype(np.int32),
                 m.data.astype(np.float64))


def _banded(n, strides):
    """Diagonally dominant, values that differ from row to row."""
    rng = np.random.default_rng(n)
    m = sp.csr_matrix((n, n))
    for s in strides:
        if s < n:
            d = -rng.uniform(0.5, 1.0, n - s)
            m = m + sp.diags([d, d], [s, -s])
    return _csr(m + sp.diags([np.asarray(abs(m).sum(axis=1)).ravel() + 0.2], [0]))


def _prec(L, prec):
    return {"fp64": (L.LD_PREC_FP64, L.LD_VT_FP64, 2), "fp32": (L.LD_PREC_MIXED, L.LD_VT_FP32, 4),
            "half": (L.LD_PREC_HALF, L.LD_VT_FP32, 8)}[prec]


def _compare(L, ctx, a, npr, prec, lanes, chunks, il, k=2):
    pr, vt, _ = _prec(L, prec)
    h = ctx.matrix(a, vt=vt)
    try:
        p = L.make_params(npr, max(1, npr // 3), 8, k, 3, precision=pr)
        got = L.ld_estimate_detail(h, p)[1]["probe_K"]
        again = L.ld_estimate_detail(h, p)[1]["probe_K"]
        L.ld_tune_set(h, p, lanes, chunks, lanes, chunks, 1, il, 0)
        ref = L.ld_estimate_detail(h, p)[1]["probe_K"]
    finally:
        ctx.release(h)
    assert np.all(np.isfinite(ref)) and np.all(ref != 0)
    assert np.array_equal(got, again)
    assert np.max(np.abs(got - ref) / np.abs(ref)) <= TOL[prec]


# block of 16-byte chunks per row: 4 lanes and 64 rows a chunk of rows (the
# latency instance up to 3072 chunks, its even grid up to twice 1536)
@pytest.mark.parametrize("chunks", [1, 7, 8, 1535, 1537, 3072, 3073])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "half"])
def test_few_chunks(L, ctx, prec, chunks):
    vec = _prec(L, prec)[2]
    a = _banded(64 * chunks - 5, (1, 37))
    for k in (2, 3):
        _compare(L, ctx, a, 4 * vec - 1, prec, 2, 2, 0, k)


# strides from 2048 rows: bands of 8 chunks, ragged planes, planes of several
# rounds, a stride longer than half the rows, the widest block
@pytest.mark.parametrize("n,strides,npr,prec,lanes,chunks", [
    (100000, (1, 32, 2048), 96, "fp32", 8, 3),
    (100001, (1, 47, 2209), 30, "fp64", 16, 1),
    (130003, (1, 2100), 30, "fp64", 16, 1),
    (130003, (1, 2047), 30, "fp64", 16, 1),
    (32401, (1, 90, 8100), 96, "fp64", 16, 3),
    (60000, (1, 31000), 64, "fp64", 32, 1),
    (250007, (1, 60, 3599, 3600, 3601), 64, "half", 8, 1),
    (120000, (1, 61, 3721), 128, "fp64", 64, 1),
])
def test_bands(L, ctx, n, strides, npr, prec, lanes, chunks):
    _compare(L, ctx, _banded(n, strides), npr, prec, lanes, chunks, 1)


# sketch widths at the padding of the factorisation's rows to 8 columns, up to
# its LDS bound of 64 and past it: the basis of two Cholesky-QR passes is
# orthonormal to the rounding of its n-term sums
@pytest.mark.parametrize("s", [1, 2, 7, 8, 9, 16, 31, 57, 63, 64, 65])
def test_sketch_basis(L, ctx, s):
    n = 900
    a = _banded(n, (1, 30))
    h = ctx.matrix(a, vt=L.LD_VT_FP64)
    try:
        p = L.make_params(s + 4, s, 8, 2, 3, precision=L.LD_PREC_FP64)
        q = L.ld_estimate_detail(h, p, n=n, basis=True)[1]["sketch_basis"]
    finally:
        ctx.release(h)
    assert q.shape == (n, s)
    assert np.max(np.abs(q.T @ q - np.eye(s))) <= 64 * n * 2.0 ** -53
