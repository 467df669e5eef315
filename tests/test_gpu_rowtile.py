"""GPU tests of the row-tile product: the row groups of a covariance-like
matrix taken 16 at a time with their union of probe rows in LDS.

Each case runs the default estimate of a matrix that keeps row groups (the
row-tile product where the block has 16 columns or more), the same estimate
with the CSR product pinned, and the CPU FP64 oracle.  The products' outputs
agree to the last bit and the fused FP64 inner products differ by their
summation order, so per-run values agree to 1e-10 with FP64 vectors; with FP32
vectors a changed last bit of a coefficient can move single entries by one
FP32 rounding (2^-24 of an entry), hence 1e-6.
"""
import numpy as np
import pytest

import oracle
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


def _scattered(n):
    return W.wendland(n, 48.0, NUG, seed=n)


MATS = {
    # scattered points: consecutive groups; less than one tile, one tile and
    # a ragged group, several tiles with a ragged last one
    "wendland_45": lambda: _scattered(45),
    "wendland_66": lambda: _scattered(66),
    "wendland_3001": lambda: _scattered(3001),
    # grids: 4 x 4 groups per tile on lines of 48, 50 and 47 rows (group lines
    # aligned or drifting), wide supports (over 320 union columns)
    "grid_40x48": lambda: W.wendland_grid(40, 48, 5.0, nugget=NUG),
    "grid_33x50": lambda: W.wendland_grid(33, 50, 3.5, nugget=NUG),
    "grid_41x47": lambda: W.wendland_grid(41, 47, 8.0, nugget=NUG),
    # entries past six rounds of 16 per group and unions too large for LDS
    "grid_30x60_wide": lambda: W.wendland_grid(30, 60, 13.0, nugget=NUG),
    # 12 tiles on 8 blocks: blocks without a tile in the second round, the last
    # tile's union beyond the columns of one load round (448 of 320)
    "grid_16x48_idle": lambda: W.wendland_grid(16, 48, 12.0, nugget=NUG),
    "dense_40x50": lambda: W.wendland_grid(40, 50, 24.0, nugget=0.5),
}


def _run(L, ctx, a, npr, s, m, k, prec, vt, method):
    nc = -(-npr // 4) * (2 if prec == L.LD_PREC_FP64 else 1)
    lanes = min(64, nc)
    h = ctx.matrix(a, vt=vt, lo_hint=NUG)
    try:
        p = L.make_params(npr, s, m, k, 5, method=method, precision=prec)
        assert L.ld_debug_row_groups(h, a.n) is not None
        default = L.ld_estimate_detail(h, p)
        pairs = []
        # the chunk mapping and the step schedule (the update or the product
        # subtracts the second-newest vector: another rounding of W, so each
        # schedule has its own reference)
        for il, sched in ((0, 1), (1, 0)):
            got = []
            for rg in (0, 1):
                L.ld_tune_set(h, p, lanes, -(-nc // lanes), lanes, -(-nc // lanes), 1, il, 0,
                              sched, rg)
                got.append(L.ld_estimate_detail(h, p))
                again = L.ld_estimate_detail(h, p)
                assert np.array_equal(again[1]["probe_K"], got[-1][1]["probe_K"])
            pairs.append(got)
    finally:
        ctx.release(h)
    return default, pairs


@pytest.mark.parametrize("name", sorted(MATS))
@pytest.mark.parametrize("npr,s,prec,vt,k,method", [
    (30, 10, "fp64", "fp64", 2, "oslq"),     # two FP64 panels of 16 columns
    (37, 9, "fp64", "fp32", 4, "oslq"),      # a last panel of 8 columns
    (16, 4, "mixed", "fp32", 2, "oslq"),     # 16 columns: one per lane
    (21, 7, "mixed", "fp32", 2, "osa_iop"),  # a panel of 24 of 32 columns; 8-column sketch runs
    (64, 20, "mixed", "fp32", 3, "oslq"),    # two panels of 32
    (70, 20, "mixed", "fp64", 12, "oslq"),   # FP64 values, two fused inner products
    (12, 4, "mixed", "fp32", 2, "oslq"),     # too narrow: the groups gather for themselves
])
def test_rowtile_against_csr_and_oracle(L, ctx, name, npr, s, prec, vt, k, method):
    a = MATS[name]()
    m = 12
    print(f"\n[case] row tiles {name} n={a.n} nnz={a.nnz} probes {npr} prec {prec} values {vt} "
          f"window {k} {method}", flush=True)
    fp64 = prec == "fp64"
    args = (npr, s, m, k, L.LD_PREC_FP64 if fp64 else L.LD_PREC_MIXED,
            L.LD_VT_FP64 if vt == "fp64" else L.LD_VT_FP32,
            L.LD_METHOD_OSLQ if method == "oslq" else L.LD_METHOD_OSA_IOP)
    (r1, _), pairs = _run(L, ctx, a, *args)
    tol = 1e-10 if fp64 else 1e-6
    for (_, d0), (_, d) in pairs:
        np.testing.assert_array_equal(d["probe_steps"], d0["probe_steps"])
        scale = np.abs(d0["probe_K"]).max()
        diff = np.abs(d["probe_K"] - d0["probe_K"]).max()
        print(f"  K differs by {diff / scale:.2e}", flush=True)
        assert diff <= tol * scale
        np.testing.assert_allclose(d["probe_norm2"], d0["probe_norm2"], rtol=1e-9)
    fn = oracle.oslq if method == "oslq" else oracle.osa_iop
    ref = fn(a, npr, s, m, k, 5, lo_hint=NUG)
    # relative to the traced sum's own scale (small matrices: terms of both signs)
    scale = max(abs(ref.logdet), np.abs(np.array(ref.probe_K)).mean() * a.n)
    assert abs(r1.logdet - ref.logdet) <= (1e-6 if fp64 else 1e-4) * scale


def test_rowtile_served_equals_alone(L):
    # batched with other widths and precisions, each result is the one it gets
    # alone (a launch's LDS class and grid do not depend on the batch)
    print("\n[case] row tiles served in batches", flush=True)
    mats = [W.wendland(5003, 48.0, NUG, seed=1), W.wendland_grid(50, 60, 6.0, nugget=NUG),
            W.wendland(2500, 30.0, NUG, seed=2), W.wendland_grid(64, 64, 3.0, nugget=NUG)]
    reqs = [(i, L.make_params(npr, 6, 14, 2, 40 + i, precision=prec))
            for i in range(4) for npr in (18, 30, 64)
            for prec in (L.LD_PREC_FP64, L.LD_PREC_MIXED)]
    with L.Context(0, max_slots=32) as c:
        hs = [c.matrix(a, vt=L.LD_VT_FP32, lo_hint=NUG) for a in mats]
        alone = [L.ld_estimate_ex(hs[i], p).logdet for i, p in reqs]
        tickets = [L.ld_submit(hs[i], p) for i, p in reqs]
        served = [L.ld_wait(c.handle, t).logdet for t in tickets]
    assert served == alone
