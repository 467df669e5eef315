"""GRF likelihood sweep (Section 4) on the GPU against the CPU oracle.

A Wendland C2 covariance Q(theta) on a small grid for several theta (support
radius theta / 10 grid spacings, nugget 1e-2 as the spectral lower bound),
a seeded smooth field x; every log-determinant (OSLQ and OSA-IOP, FP64)
within 1e-6 of the oracle, x^T Q x within 1e-12, L(theta) assembled alike,
and the swept requests (in flight together) equal to the same requests run
alone.  The paper's values need its field and theta units and are not
reproduced (parity unpinned for those).
"""
import math

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2606_07004_amd import liblogdet
    liblogdet.lib()
    return liblogdet


def _mat(theta, ny=24, nx=30):
    return W.wendland_grid(ny, nx, W.grf_rho(theta), nugget=1e-2)


@pytest.mark.parametrize("method", ["oslq", "osa_iop"])
def test_grf_sweep_matches_oracle(L, method):
    from paper_2606_07004_amd import grf
    print(f"\n[case] grf sweep {method} 24x30 thetas 20,40,60", flush=True)
    thetas = (20, 40, 60)
    x = W.grf_field(24, 30, seed=7)
    if method == "oslq":
        p = L.make_params(30, 10, 40, 2, 1, method=L.LD_METHOD_OSLQ)
    else:
        p = L.make_params(21, 7, 20, 2, 1, method=L.LD_METHOD_OSA_IOP, tol=1e-6)
    with L.Context(0, max_slots=4) as c:
        recs = grf.theta_sweep(c, thetas, _mat, x, p, lo_hint=lambda th: 1e-2)
        alone = []
        for th in thetas:
            h = c.matrix(_mat(th), lo_hint=1e-2)
            alone.append(L.ld_estimate_ex(h, p).logdet)
            c.release(h)
    for rec, th, al in zip(recs, thetas, alone):
        a = _mat(th)
        if method == "oslq":
            ref = oracle.oslq(a, 30, 10, 40, 2, 1, lo_hint=1e-2)
        else:
            ref = oracle.osa_iop(a, 21, 7, 20, 2, 1, lo_hint=1e-2, tol=1e-6)
        q = sp.csr_matrix((a.values, a.col_idx, a.row_ptr), shape=(a.n, a.n))
        quad = float(x @ (q @ x))
        ll = 0.5 * ref.logdet - 0.5 * quad - 0.5 * a.n * math.log(2 * math.pi)
        rel = abs(rec["logdet"] - ref.logdet) / abs(ref.logdet)
        print(f"  theta {th}: logdet {rec['logdet']:.10g} oracle {ref.logdet:.10g} rel {rel:.2e} "
              f"loglik {rec['loglik']:.8g}", flush=True)
        assert rel <= 1e-6
        assert rec["quad"] == pytest.approx(quad, rel=1e-12)
        assert rec["loglik"] == pytest.approx(ll, rel=1e-6, abs=1e-6 * abs(ref.logdet))
        assert rec["logdet"] == al  # batched sweep == alone, bitwise


def test_quad_form_ragged(L):
    print("\n[case] quad form ragged n", flush=True)
    a = W.er_laplacian(5003, 20000, seed=9)
    x = np.random.default_rng(2).standard_normal(a.n)
    q = sp.csr_matrix((a.values, a.col_idx, a.row_ptr), shape=(a.n, a.n))
    with L.Context(0) as c:
        h = c.matrix(a)
        got = L.ld_quad_form(h, x)
        c.release(h)
    assert got == pytest.approx(float(x @ (q @ x)), rel=1e-12)


@pytest.mark.parametrize("name", ["one", "diag", "lap2d", "grid", "long_rows", "ragged"])
def test_quad_form_shapes(L, name):
    # lanes per row from 2 (short rows) to 64 (rows of 500 entries), rows
    # without a full group of four entries per lane, one row, more rows than
    # one pass of the grid
    rng = np.random.Generator(np.random.PCG64(3))
    a = {"one": lambda: W.diag_matrix([2.5]),
         "diag": lambda: W.diag_matrix(rng.uniform(1, 2, 70001)),
         "lap2d": lambda: W.lap2d(411, 0.1),
         "grid": lambda: W.wendland_grid(37, 41, 5.0),
         "long_rows": lambda: W.from_dense(W.random_spd_dense(501, 5)),
         "ragged": lambda: W.er_laplacian(1003, 9000, seed=4)}[name]()
    x = rng.standard_normal(a.n)
    print(f"\n[case] quad form {name} n={a.n} nnz={a.nnz}", flush=True)
    with L.Context(0) as c:
        h = c.matrix(a)
        est = L.ld_estimate_ex(h, L.make_params(8, 2, 1, 1, 7)) if a.n > 1 else None
        got = L.ld_quad_form(h, x)
        assert L.ld_quad_form(h, x) == got  # a fixed summation order
        if est is not None:  # the shared workspace leaves estimates alone
            assert L.ld_estimate_ex(h, L.make_params(8, 2, 1, 1, 7)).logdet == est.logdet
    q = a.to_scipy().astype(np.longdouble)
    xl = x.astype(np.longdouble)
    want = float(xl @ (q @ xl))
    # about 100 roundings (2^-53 each) of partial sums bounded by sum |x_i a_ij x_j|
    bound = float(np.abs(x) @ (abs(a.to_scipy()) @ np.abs(x)))
    assert abs(got - want) <= 1e-13 * bound


def test_quad_form_keeps_captured_estimates(L):
    # a quadratic form larger than the estimates' workspace leaves the captured
    # graphs alone: the next estimate of the small matrix is a replay
    print("\n[case] quad form beside a captured estimate", flush=True)
    small, large = W.lap2d(24, 0.1), W.diag_matrix(np.full(3_000_000, 2.0))
    with L.Context(0) as c:
        hs, hl = c.matrix(small), c.matrix(large)
        p = L.make_params(8, 2, 10, 2, 7)
        assert L.ld_request_bytes(hs, p) < 8 * large.n
        first = [L.ld_estimate_ex(hs, p).logdet for _ in range(3)]
        before = L.ld_graph_stats_get(c.handle)
        assert before.replays >= 1 and before.cached == 1
        assert L.ld_quad_form(hl, np.ones(large.n)) == 2.0 * large.n
        again = L.ld_estimate_ex(hs, p).logdet
        after = L.ld_graph_stats_get(c.handle)
        assert (after.captures, after.cached) == (before.captures, 1)
        assert after.replays == before.replays + 1
        assert first == [again] * 3
        # the form's buffer goes with the last matrix and comes back
        c.release(hs)
        c.release(hl)
        hl = c.matrix(large)
        assert L.ld_quad_form(hl, np.ones(large.n)) == 2.0 * large.n
