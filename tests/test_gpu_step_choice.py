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
    (20000, 8, "fp64", "fp64", 2, 1), (20000, 64, "half", "fp32", 2, 1),
    (20000, 12, "mixed", "fp32", 2, 1), (256 * 512, 4, "mixed", "fp32", 2, 0),
    (256 * 512 + 1, 4, "mixed", "fp32", 2, 1), (128 * 512 + 1, 4, "fp64", "fp64", 2, 1),
    (64 * 2048, 30, "half", "fp32", 2, 0), (64 * 2048 + 1, 30, "half", "fp32", 2, 1),
    (64 * 3072 + 1, 30, "half", "fp32", 2, 0), (32 * 640, 64, "half", "fp32", 2, 1),
    (32 * 640 + 1, 64, "half", "fp32", 2, 0), (16 * 640, 124, "half", "fp64", 2, 1),
    (64 * 640, 30, "half", "fp64", 2, 0), (32 * 1612, 64, "half", "fp64", 2, 0),
    (32 * 1612 + 1, 64, "half", "fp64", 2, 1), (32 * 2150, 64, "half", "fp64", 2, 1),
    (32 * 2150 + 1, 64, "half", "fp64", 2, 0),
])
def test_latency_instance(L, ctx, n, npr, prec, vt, k, latency):
    got = _paths(L, ctx, _stripes(n, (1, 37)), npr, prec, vt, k)
    assert got["product"] == 0 and got["latency"] == latency


# the update that reads a row ahead: rows of less than a line (7 chunks and
# fewer) up to 320 chunks of rows, FP16 ones past 1024 again, with two to four
# vectors those of 4 columns up to 1024 chunks; wider rows up to 24
# (12) rounds of 2048 chunks
@pytest.mark.parametrize("n,npr,prec,k,ahead", [
    (256 * 320, 4, "mixed", 2, 1), (256 * 320 + 1, 4, "mixed", 2, 0),
    (32 * 320, 28, "mixed", 2, 1), (32 * 320 + 1, 28, "mixed", 2, 0),
    (32 * 320 + 1, 30, "mixed", 2, 1), (256 * 320 + 1, 2, "fp64", 2, 0),
    (128 * 1024, 4, "fp64", 4, 1), (128 * 1024 + 1, 4, "fp64", 4, 0),
    (256 * 1024, 4, "mixed", 3, 1), (256 * 1024 + 1, 4, "mixed", 3, 0),
    (256 * 1024 + 1, 4, "mixed", 4, 1), (64 * 1024 + 1, 8, "fp64", 4, 1),
    (64 * 320 + 1, 30, "half", 2, 0), (64 * 1024 + 1, 30, "half", 2, 1),
    (16 * 24 * 2048, 64, "mixed", 2, 1), (16 * 24 * 2048 + 1, 64, "mixed", 2, 0),
    (16 * 12 * 2048, 30, "fp64", 4, 1), (16 * 12 * 2048 + 1, 30, "fp64", 4, 0),
    (16 * 12 * 2048 + 1, 30, "fp64", 2, 1), (3000, 30, "mixed", 6, 0),
])
def test_update_ahead(L, ctx, n, npr, prec, k, ahead):
    assert _paths(L, ctx, _stripes(n, (1,)), npr, prec, k=k)["update_ahead"] == ahead


# row groups in their default geometry (one chunk per lane, FP64 vectors two) are
# the row tiles, other lanes and chunks the row-group product; per-probe values
# against the CSR product in the same step schedule: each row's sum is the same
# chain of multiply-adds, the fused FP64 inner products differ by their order, and
# FP32 vectors by single roundings of 2^-24 after them
@pytest.mark.parametrize("npr,prec,vt,k,lanes,chunks,product", [
    (30, "mixed", "fp32", 2, 8, 1, 2), (30, "mixed", "fp32", 2, 4, 2, 1),
    (30, "mixed", "fp32", 2, 16, 1, 1), (22, "mixed", "fp32", 12, 3, 2, 1),
    (30, "fp64", "fp64", 2, 8, 2, 2), (30, "fp64", "fp64", 12, 8, 2, 2),
    (37, "fp64", "fp32", 4, 10, 2, 2), (30, "fp64", "fp64", 2, 16, 1, 1),
    (16, "mixed", "fp64", 2, 4, 1, 2), (16, "mixed", "fp64", 12, 4, 1, 2),
    (13, "mixed", "fp64", 3, 2, 2, 1), (12, "mixed", "fp32", 2, 3, 1, 1),
])
@pytest.mark.parametrize("il", [0, 1])
def test_row_group_choices(L, ctx, npr, prec, vt, k, lanes, chunks, product, il):
    a = W.wendland(3001, 48.0, NUG, seed=5)
    h = ctx.matrix(a, vt=L.LD_VT_FP64 if vt == "fp64" else L.LD_VT_FP32, lo_hint=NUG)
    try:
        p = L.make_params(npr, 4, 14, k, 7,
                          precision=L.LD_PREC_FP64 if prec == "fp64" else L.LD_PREC_MIXED)
        print(f"\n[case] row groups pinned: probes {npr} {prec} values {vt} window {k} "
              f"{lanes} x {chunks} interleave {il}", flush=True)
        K = []
        for rg in (0, 1):
            L.ld_tune_set(h, p, lanes, chunks, lanes, chunks, 1, il, 0, 1, rg)
            got = L.ld_debug_step_paths(h, p)
            assert (got["product"], got["lanes"], got["chunks"]) == (product if rg else 0, lanes,
                                                                     chunks)
            K.append(L.ld_estimate_detail(h, p)[1]["probe_K"])
            assert np.array_equal(L.ld_estimate_detail(h, p)[1]["probe_K"], K[-1])
    finally:
        ctx.release(h)
    assert np.abs(K[1] - K[0]).max() <= (1e-10 if prec == "fp64" else 1e-6) * np.abs(K[0]).max()


# the tuner times the untuned geometries and reports their times: an untuned
# choice that its list lacked (5 chunks of an update: 8 lanes) or that came last
# (tiles, against the CSR rows' time) made a tuned matrix slower than an untuned
@pytest.mark.parametrize("npr,prec,vt", [(20, "mixed", "fp32"), (100, "fp64", "fp64"),
                                         (128, "fp64", "fp64"), (18, "mixed", "bf16")])
def test_tuner_times_the_default(L, ctx, npr, prec, vt):
    a = W.wendland(20011, 48.0, NUG, seed=5)
    h = ctx.matrix(a, vt={"fp64": L.LD_VT_FP64, "fp32": L.LD_VT_FP32, "bf16": L.LD_VT_BF16}[vt],
                   lo_hint=NUG)
    try:
        p = L.make_params(npr, 4, 14, 2, 7,
                          precision=L.LD_PREC_FP64 if prec == "fp64" else L.LD_PREC_MIXED)
        untuned = L.ld_debug_step_paths(h, p)
        print(f"\n[case] tuner probes {npr} {prec} values {vt} untuned {untuned}", flush=True)
        tr = L.ld_autotune(h, p, 5)
        tuned = L.ld_debug_step_paths(h, p)
        print("  ", tr.as_dict(), tuned, flush=True)
        # the tile product is far ahead of every other one here (0.6 of the CSR
        # product's time and less), so the tuner has to find it
        assert untuned["product"] == tuned["product"] == (0 if vt == "bf16" else 2)
        assert tr.spmm_ms <= tr.spmm_default_ms and tr.update_ms <= tr.update_default_ms
        assert tr.spmm_row_groups == (0 if vt == "bf16" else 1)
        # what the tuner reports can be set again
        L.ld_tune_set(h, p, tr.spmm_lanes, tr.spmm_chunks, tr.update_lanes, tr.update_chunks,
                      tr.spmm_entry_split, tr.spmm_interleave, tr.spmm_row_stride, tr.step_presub,
                      tr.spmm_row_groups)
        assert L.ld_debug_step_paths(h, p) == tuned
    finally:
        ctx.release(h)


def _dofs(graph, b):
    """b unknowns per node of a graph Laplacian: dense b x b blocks."""
    return _csr(sp.kron(graph.to_scipy(), np.eye(b) * 2 + 0.5, format="csr"))


# the row groups' default is their tiles where these pay, by the blocks per CU that
# the largest union leaves, the rounds of blocks and what neighbouring tiles share.
# One block (1000 tiles of a random graph, 3.9 rounds per panel; 312 tiles, 1.2; a
# covariance of 190 entries per row, 4.2), two blocks (2813 tiles, 5.5 rounds per
# panel; 375 tiles), three, and a few large unions
@pytest.mark.parametrize("name,npr,prec,vt,product", [
    ("random_1", 32, "mixed", "fp32", 2), ("random_1", 33, "mixed", "fp32", 1),
    ("random_1", 96, "mixed", "fp32", 1), ("random_1", 24, "fp64", "fp64", 2),
    ("random_1", 48, "fp64", "fp64", 2), ("random_1", 49, "fp64", "fp64", 1),
    ("random_1", 64, "mixed", "fp64", 2), ("random_1", 65, "mixed", "fp64", 0),
    ("random_1s", 128, "mixed", "fp32", 2), ("random_1s", 128, "fp64", "fp64", 2),
    ("random_2", 64, "mixed", "fp32", 2), ("random_2", 65, "mixed", "fp32", 1),
    ("random_2", 33, "fp64", "fp64", 1), ("random_2s", 128, "fp64", "fp64", 2),
    ("random_3", 128, "mixed", "fp32", 2), ("random_16", 128, "mixed", "fp64", 2),
    ("random_big", 64, "fp64", "fp64", 1), ("random_big", 32, "fp64", "fp64", 2),
    ("wide", 32, "mixed", "fp32", 2), ("wide", 33, "mixed", "fp32", 1),
    ("wide", 96, "mixed", "fp32", 2), ("wide", 128, "mixed", "fp32", 1),
    ("wide", 48, "fp64", "fp64", 2), ("wide", 49, "fp64", "fp64", 1),
    ("wide", 128, "mixed", "fp64", 2), ("hub", 64, "mixed", "fp32", 2),
    ("hub", 64, "fp64", "fp64", 2),
])
def test_tiles_where_they_pay(L, ctx, name, npr, prec, vt, product):
    def hub():
        a = W.wendland(100000, 48.0, NUG, seed=1).to_scipy().tolil()
        cols = np.arange(0, 100000, 125)
        a[7000, cols] = a[7000, cols].toarray() + 1e-4
        a[cols, 7000] = a[cols, 7000].toarray() + 1e-4
        return _csr(a)
    a = {"random_1": lambda: _dofs(W.er_laplacian(16000, 16000 * 5, seed=1), 4),
         "random_1s": lambda: _dofs(W.er_laplacian(5000, 5000 * 5, seed=1), 4),
         "random_2": lambda: _dofs(W.er_laplacian(45000, 45000 * 5 // 2, seed=1), 4),
         "random_2s": lambda: _dofs(W.er_laplacian(6000, 6000 * 5 // 2, seed=1), 4),
         "random_3": lambda: _dofs(W.er_laplacian(6000, 6000 * 1, seed=1), 4),
         "random_16": lambda: _dofs(W.er_laplacian(2000, 2000 * 3, seed=1), 16),
         "random_big": lambda: _dofs(W.er_laplacian(140000, 140000, seed=1), 4),
         "wide": lambda: W.wendland_grid(230, 300, 8.0, nugget=NUG), "hub": hub}[name]()
    got = _paths(L, ctx, a, npr, prec, vt, lo=1e-2)
    print(f"  {got}", flush=True)
    blocks = {"random_1": 1, "random_1s": 1, "random_16": 1, "random_2": 2, "random_2s": 2,
              "wide": 1, "hub": 1}.get(name, 3)
    rows = {1: (633, 1248), 2: (413, 632), 3: (1, 412)}[blocks]  # of 128 bytes in 52.5 and 80 KB
    assert rows[0] <= got["tile_union"] <= rows[1] and got["product"] == product


# bands: strides from 2048 rows and 8 chunks of rows per band on, whole runs of the
# stride but for 2% of the rows (60 runs less 40 or 1200 rows, 2.1 runs), more rows
# than the latency instance takes, and not where rows of up to 256 bytes make a run
# a multiple of 4 MB
@pytest.mark.parametrize("n,strides,npr,prec,bands", [
    (100 * 2048, (1, 32, 2048), 96, "mixed", 1), (100 * 2047, (1, 32, 2047), 96, "mixed", 0),
    (60 * 2500 - 40, (1, 50, 2500), 96, "mixed", 1), (60 * 2500 - 1200, (1, 50, 2500), 96, "mixed", 1),
    (10 * 15000 - 1200, (1, 50, 15000), 96, "mixed", 1),
    (10 * 15000 - 4000, (1, 50, 15000), 96, "mixed", 0),
    (21 * 7000, (1, 50, 70000), 96, "mixed", 0), (2 * 70000, (1, 50, 70000), 96, "mixed", 1),
    (20 * 2048, (1, 32, 2048), 30, "mixed", 0), (120 * 4096, (1, 50, 4096), 8, "fp64", 1),
    (120 * 4095, (1, 50, 4095), 8, "fp64", 0), (60 * 2048, (1, 50, 2048), 5, "half", 0),
    (16 * 16384, (1, 128, 16384), 64, "mixed", 0), (16 * 16384, (1, 128, 16384), 60, "mixed", 1),
    (16 * 16384, (1, 128, 16384), 68, "mixed", 1), (16 * 16384, (1, 128, 16384), 128, "mixed", 1),
    (16 * 16384, (1, 128, 16384), 30, "fp64", 0), (16 * 16400, (1, 128, 16400), 64, "mixed", 1),
])
def test_bands_of_whole_runs(L, ctx, n, strides, npr, prec, bands):
    assert _paths(L, ctx, _stripes(n, strides), npr, prec)["bands"] == bands


# values at the sizes where the rules above change, against the step with two
# chunks per lane (another product and another update): each row's sums are the
# same chains of multiply-adds, the FP64 sums of inner products differ by their
# order (1e-10), FP32 and FP16 vectors by single roundings of 2^-24 and 2^-11
# after them (1e-6, 5e-4)
@pytest.mark.parametrize("n,npr,prec,vt,k", [
    (16 * 24 * 2048 + 1, 64, "mixed", "fp32", 2), (16 * 24 * 2048, 64, "mixed", "fp32", 3),
    (16 * 12 * 2048 + 1, 30, "fp64", "fp64", 4), (256 * 320 + 1, 4, "mixed", "fp32", 2),
    (128 * 320 + 1, 4, "fp64", "fp64", 3), (64 * 320 + 1, 30, "half", "fp32", 2),
    (64 * 1024 + 1, 30, "half", "fp32", 2), (16 * 3072 + 1, 30, "fp64", "fp64", 10),
    (16 * 3072, 30, "fp64", "fp64", 10), (32 * 3072, 30, "mixed", "fp64", 2),
    (20011, 8, "mixed", "fp64", 2), (20011, 60, "half", "fp32", 2),
    (128 * 512 + 1, 8, "mixed", "fp32", 2), (64 * 2048 + 1, 30, "half", "fp32", 2),
    (32 * 1612 + 1, 64, "half", "fp64", 2), (16 * 640, 124, "half", "fp32", 2),
])
def test_values_where_rules_change(L, ctx, n, npr, prec, vt, k):
    a = _stripes(n, (1, 37))
    a.values[a.col_idx == np.repeat(np.arange(n), np.diff(a.row_ptr))] += \
        np.random.default_rng(n).uniform(0, 1, n)
    vec = {"fp64": 2, "mixed": 4, "half": 8}[prec]
    nc = -(-npr // vec) if prec == "half" else -(-npr // 4) * (4 // vec)
    h = ctx.matrix(a, vt=L.LD_VT_FP64 if vt == "fp64" else L.LD_VT_FP32)
    try:
        p = L.make_params(npr, max(1, npr // 3), 12, k, 3, precision={
            "fp64": L.LD_PREC_FP64, "mixed": L.LD_PREC_MIXED, "half": L.LD_PREC_HALF}[prec])
        print(f"\n[case] values n={n} probes {npr} {prec} values {vt} window {k} "
              f"{L.ld_debug_step_paths(h, p)}", flush=True)
        got = L.ld_estimate_detail(h, p)[1]["probe_K"]
        L.ld_tune_set(h, p, -(-nc // 2), 2, -(-nc // 2), 2)
        ref = L.ld_estimate_detail(h, p)[1]["probe_K"]
    finally:
        ctx.release(h)
    assert np.all(np.isfinite(ref)) and np.all(ref != 0)
    tol = {"fp64": 1e-10, "mixed": 1e-6, "half": 5e-4}[prec]
    assert np.max(np.abs(got - ref) / np.abs(ref)) <= tol
