"""Galerkin patterns, transposes and launch shapes formed on the device, at the edges of
their row forms: short rows, rows that overflow the first hash tables, rows beyond the
largest (sorted instead), long rows of R, rows with no entries in P."""
import gc

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from tests.gpu_util import T, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


def spd_from(n, i, j, seed):
    """Symmetric strictly dominant matrix with couplings (i, j)."""
    g = np.random.default_rng(seed)
    W = sp.coo_matrix((-g.uniform(0.1, 1.0, len(i)), (i, j)), shape=(n, n))
    W = (W + W.T).tocsr()
    W.setdiag(0)
    W.eliminate_zeros()
    A = (W + sp.diags(1.0 - np.asarray(W.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return A


def transfer(n, nc, per_row, seed, empty=0):
    """P with per_row random coarse columns per fine row (the first `empty` rows have none),
    every coarse column used."""
    g = np.random.default_rng(seed)
    rows = np.concatenate([np.repeat(np.arange(empty, n), per_row), empty + np.arange(nc) % (n - empty)])
    cols = np.concatenate([g.integers(0, nc, (n - empty) * per_row), np.arange(nc)])
    P = sp.coo_matrix((np.ones(len(rows)), (rows, cols)), shape=(n, nc)).tocsr()
    P.data[:] = g.uniform(0.2, 1.0, P.nnz)
    P.sort_indices()
    return P


CASES = {
    # name: (n, coupling builder, coarse sizes, columns per P row)
    "chain": (700, lambda n, g: (np.arange(n - 1), np.arange(1, n)), [90], 1),
    "one_row_blocks": (257, lambda n, g: (np.arange(n - 1), np.arange(1, n)), [16], 3),
    "dense_graph": (900, lambda n, g: (g.integers(0, n, 40 * n), g.integers(0, n, 40 * n)), [300], 4),
    # one row coupled to everything: its A P row has more columns than the others by far
    "hub": (6000, lambda n, g: (np.concatenate([np.arange(n - 1), np.zeros(n - 1, int)]),
                                np.concatenate([np.arange(1, n), np.arange(1, n)])), [3000, 200], 1),
    # ... and beyond the largest table
    "big_hub": (24000, lambda n, g: (np.concatenate([np.arange(n - 1), np.zeros(n - 1, int)]),
                                     np.concatenate([np.arange(1, n), np.arange(1, n)])), [12000, 150], 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_product_patterns(name):
    from paper_2108_02054_amd import AMG
    n, couple, sizes, per_row = CASES[name]
    i, j = couple(n, np.random.default_rng(1))
    A = spd_from(n, i, j, 2)
    Ps, m = [], n
    for l, nc in enumerate(sizes):
        Ps.append(transfer(m, nc, per_row, 10 + l, empty=3 if name == "dense_graph" else 0))
        m = nc
    print(f"case product patterns {name}: n={n} longest row {np.diff(A.indptr).max()}", flush=True)
    args = [(T(P.indptr.astype(np.int32)), T(P.indices.astype(np.int32)), T(P.data), P.shape[1]) for P in Ps]
    g = AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data), transfer=args)
    for scale in (1.0, 2.5):
        if scale != 1.0:
            g.rebuild(T(scale * A.data))
        B = (scale * A).tocsr()
        for l, P in enumerate(Ps):
            # structural pattern: every product term makes an entry
            one = lambda M: sp.csr_matrix((np.ones(M.nnz), M.indices, M.indptr), shape=M.shape)  # noqa: E731
            C = (P.T @ B @ P).tocsr()
            S = (one(P).T @ one(B) @ one(P)).tocsr()
            S.sort_indices()
            got = g.level(l + 1)["A"]
            assert np.array_equal(got[0], S.indptr) and np.array_equal(got[1], S.indices)
            D = sp.csr_matrix((got[2], got[1], got[0]), shape=C.shape)
            # sums of at most 2e5 rounded products of one sign pattern: well below 1e-12
            assert abs(D - C).max() <= 1e-12 * abs(C).max()
            B = sp.csr_matrix((got[2], got[1], got[0]), shape=C.shape)
    f = np.random.default_rng(3).uniform(-1, 1, n)
    z = g.vcycle(T(f)).cpu().numpy()
    assert np.isfinite(z).all() and np.abs(z).max() > 0
    g.close()


@pytest.mark.parametrize("rows,per_row,couplings,span", [
    (5, 1, 3, 5), (60, 2, 6, 9), (1024, 2, 5, 30), (1025, 2, 5, 30), (4096, 3, 4, 40), (4097, 3, 4, 40),
    (300, 12, 40, 120), (300, 30, 60, 240), (2000, 12, 30, 130), (2000, 20, 50, 250)])
def test_small_products_match_position_map(monkeypatch, rows, per_row, couplings, span):
    """The small products' owner form (a workgroup per row, G lanes per row; 8 to 248 columns
    in a row) against the position-map form, bit for bit, in FP64 and FP32."""
    from paper_2108_02054_amd import AMG
    g = np.random.default_rng(rows)
    n, mid = 6 * rows, rows
    near = lambda a, d, m: np.clip(a + g.integers(-d, d + 1, len(a)), 0, m - 1)  # noqa: E731
    i = np.repeat(np.arange(n), 3)
    A = spd_from(n, i, near(i, 8, n), 3)
    agg = np.arange(n) // 6
    r = np.repeat(np.arange(n), per_row)
    P0 = sp.coo_matrix((np.ones(len(r) + n), (np.r_[r, np.arange(n)], np.r_[near(agg[r], span // 4, mid), agg])),
                       shape=(n, mid)).tocsr()
    P0.data[:] = g.uniform(0.2, 1.0, P0.nnz)
    P0.sort_indices()
    nc = max(2, mid // 3)
    agg1 = np.arange(mid) * nc // mid
    r = np.repeat(np.arange(mid), 2)
    P1 = sp.coo_matrix((np.ones(len(r) + mid), (np.r_[r, np.arange(mid)], np.r_[near(agg1[r], max(1, span // 8), nc), agg1])),
                       shape=(mid, nc)).tocsr()
    P1.data[:] = g.uniform(0.2, 1.0, P1.nnz)
    P1.sort_indices()
    args = lambda: [(T(P.indptr.astype(np.int32)), T(P.indices.astype(np.int32)), T(P.data), P.shape[1])  # noqa: E731
                    for P in (P0, P1)]
    print(f"case owner form rows={rows} per_row={per_row} span={span}", flush=True)
    for precision in (0, 1):
        got = []
        for form in (None, "pos"):
            if form:
                monkeypatch.setenv("AMGMI_GALERKIN", form)
            else:
                monkeypatch.delenv("AMGMI_GALERKIN", raising=False)
            h = AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data), transfer=args(),
                    precision=precision, smoother=rows % 2, coarse_enough=2048)
            h.rebuild(T(1.25 * A.data))
            got.append([h.level(l) for l in range(3)])
            h.close()
        for a, b in zip(*got):
            assert np.array_equal(a["A"][2], b["A"][2])
            assert a["m"] is None or np.array_equal(a["m"], b["m"])


def test_v_cycle_of_long_restriction_rows():
    """One aggregate of 5000 rows: its row of R is longer than the ranked transpose takes."""
    from paper_2108_02054_amd import AMG
    n = 7000
    A = spd_from(n, np.arange(n - 1), np.arange(1, n), 4)
    agg = np.where(np.arange(n) < 5000, 0, 1 + (np.arange(n) - 5000) // 20)
    P = sp.csr_matrix((np.ones(n), agg, np.arange(n + 1)), shape=(n, agg.max() + 1))
    print("case long restriction row", flush=True)
    g = AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data),
            transfer=[(T(P.indptr.astype(np.int32)), T(P.indices.astype(np.int32)), T(P.data), P.shape[1])])
    # the two-level V-cycle with one Jacobi sweep before and after, in dense arithmetic
    f = np.random.default_rng(5).uniform(-1, 1, n)
    m = 0.72 / A.diagonal()
    u = m * f
    uc = np.linalg.solve((P.T @ A @ P).toarray(), P.T @ (f - A @ u))
    u = u + P @ uc
    u = u + m * (f - A @ u)
    # condition of the coarse operator below 1e4: its solve is good to 1e4 eps
    assert rel_max(g.vcycle(T(f)).cpu().numpy(), u) <= 1e-10
    g.close()


@pytest.mark.parametrize("n,nc,per_row", [
    (5000, 4000, 2),    # rows of R of a few entries
    (20000, 300, 1),    # ... of about 70, in more rows than lanes are short of
    (4000, 40, 6),      # ... of hundreds, in few rows
    (2400, 5, 4),       # ... up to the longest that is ranked
    (3000, 1500, 30),   # more distinct columns under a workgroup than its table holds
    (255, 70, 3), (257, 33, 5)])
def test_transpose_by_ranks(n, nc, per_row):
    """R = P^T through the product that reads it: pattern exact, values to rounding."""
    from paper_2108_02054_amd import AMG
    A = spd_from(n, np.arange(n - 1), np.arange(1, n), 6)
    P = transfer(n, nc, per_row, 21, empty=2)
    P2 = transfer(nc, min(nc, 30), 1, 22)
    print(f"case transpose n={n} nc={nc} longest row of R {np.bincount(P.indices).max()}", flush=True)
    args = [(T(M.indptr.astype(np.int32)), T(M.indices.astype(np.int32)), T(M.data), M.shape[1]) for M in (P, P2)]
    g = AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data), transfer=args)
    one = lambda M: sp.csr_matrix((np.ones(M.nnz), M.indices, M.indptr), shape=M.shape)  # noqa: E731
    S = (one(P).T @ one(A) @ one(P)).tocsr()
    S.sort_indices()
    C = (P.T @ A @ P).tocsr()
    got = g.level(1)["A"]
    assert np.array_equal(got[0], S.indptr) and np.array_equal(got[1], S.indices)
    D = sp.csr_matrix((got[2], got[1], got[0]), shape=C.shape)
    # at most 2400 * 3 products per entry, rounded one by one
    assert abs(D - C).max() <= 1e-12 * abs(C).max()
    g.close()


@pytest.mark.parametrize("kind,n", [("27pt", 41), ("27pt", 40), ("27pt", 19), ("7pt", 41), ("dense", 1500)])
def test_aggregates_by_row_lanes(kind, n):
    """MIS-2 and the aggregation passes with 8 lanes per row (68921 rows of 27 entries), 32 (as
    many as 64000, and few long rows) and one: aggregates as the oracle's, on every level."""
    from tests.gpu_util import both, compare_levels
    from workloads import lognormal_27pt, two_fluid_7pt
    if kind == "dense":
        g = np.random.default_rng(8)
        A = spd_from(n, g.integers(0, n, 60 * n), g.integers(0, n, 60 * n), 9)
        p, c, v = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    else:
        p, c, v = lognormal_27pt(n, 1) if kind == "27pt" else two_fluid_7pt(n, 0.4)
    print(f"case row lanes {kind} {n}", flush=True)
    g, o = both(p, c, v, coarse_enough=20)
    compare_levels(g, o, tol=1e-10, values=False)
    g.close()
    o.close()


@pytest.mark.parametrize("n,nc,couplings,per_row", [
    (3000, 2048, 25, 3), (3000, 2049, 25, 3),  # the most rows that share wavefronts, and one more
    (900, 70, 20, 2),                           # C rows of fewer columns than a byte holds
    (1500, 1200, 60, 1),                        # rows of R of one or two entries: idle wavefronts
    (700, 500, 120, 6)])
def test_product_rows_by_several_wavefronts(n, nc, couplings, per_row):
    """Products of few rows with many terms each: patterns exact, values to rounding, as set up
    and after a partial update (which walks the plan)."""
    from paper_2108_02054_amd import AMG
    g = np.random.default_rng(n + nc)
    A = spd_from(n, g.integers(0, n, couplings * n), g.integers(0, n, couplings * n), 12)
    P, P2 = transfer(n, nc, per_row, 31, empty=1), transfer(nc, min(nc, 40), 1, 32)
    args = [(T(M.indptr.astype(np.int32)), T(M.indices.astype(np.int32)), T(M.data), M.shape[1]) for M in (P, P2)]
    print(f"case several wavefronts n={n} nc={nc} couplings={couplings}", flush=True)
    h = AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data), transfer=args)
    one = lambda M: sp.csr_matrix((np.ones(M.nnz), M.indices, M.indptr), shape=M.shape)  # noqa: E731
    S1 = (one(P).T @ one(A) @ one(P)).tocsr()
    S2 = (one(P2).T @ one(S1) @ one(P2)).tocsr()
    for scale in (1.0, 1.5):
        if scale != 1.0:
            h.rebuild(T(scale * A.data))
        B = (scale * A).tocsr()
        for l, (Q, S) in enumerate(((P, S1), (P2, S2))):
            S.sort_indices()
            C = (Q.T @ B @ Q).tocsr()
            got = h.level(l + 1)["A"]
            assert np.array_equal(got[0], S.indptr) and np.array_equal(got[1], S.indices)
            B = sp.csr_matrix((got[2], got[1], got[0]), shape=C.shape)
            # sums of at most 1e6 rounded products: well below 1e-11 of the largest entry
            assert abs(B - C).max() <= 1e-11 * abs(C).max()
    h.close()


@pytest.mark.parametrize("N", [97, 98, 104])  # 32633, 33633 and 39929 rows on level 1
def test_products_of_long_rows_two_terms_per_lane(monkeypatch, N):
    """Two B terms per lane and entry from 32768 rows of 44 entries on: the coarse operators of
    an update equal those of one term per lane bit for bit."""
    from paper_2108_02054_amd import AMG
    from workloads import lognormal_27pt
    p, c, v = lognormal_27pt(N, 0)
    v1 = 1.25 * v
    print(f"case two terms per lane N={N}", flush=True)
    got = []
    for form in (None, "pos:16:1"):
        if form:
            monkeypatch.setenv("AMGMI_GALERKIN", form)
        g = AMG(T(p), T(c), T(v), eps_strong=0.02)
        g.rebuild(T(v1))
        got.append([g.level(l)["A"][2] for l in range(1, g.num_levels)])
        g.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


# on level 1 a workgroup per row up to 1024 rows, G lanes per row up to 4096; rows of 8 to 248
# columns (8, 16, 32 and 64 lanes; one, two and four positions per lane)
@pytest.mark.parametrize("rows,per_row,couplings,span", [
    (60, 2, 6, 9), (300, 3, 6, 20), (300, 12, 40, 120), (300, 30, 60, 240), (1024, 2, 5, 30),
    (1025, 2, 5, 30), (2000, 12, 30, 130), (4096, 3, 4, 40)])
@pytest.mark.parametrize("precision", [0, 1])
def test_owner_form_correction(monkeypatch, rows, per_row, couplings, span, precision):
    """Q = (I - M A) P as the owner form writes it, through the V-cycle that reads it: bit for
    bit the position-map form's.  (The form is demanded: another one would be an error.)"""
    from paper_2108_02054_amd import AMG
    g = np.random.default_rng(rows + span)
    n, mid = 6 * rows, rows
    near = lambda a, d, m: np.clip(a + g.integers(-d, d + 1, len(a)), 0, m - 1)  # noqa: E731
    A = spd_from(n, np.repeat(np.arange(n), 3), near(np.repeat(np.arange(n), 3), 8, n), 3)

    def spread(n, nc, per_row, reach):
        agg = np.arange(n) * nc // n
        r = np.repeat(np.arange(n), per_row)
        P = sp.coo_matrix((np.ones(len(r) + n), (np.r_[r, np.arange(n)], np.r_[near(agg[r], reach, nc), agg])),
                          shape=(n, nc)).tocsr()
        P.data[:] = g.uniform(0.2, 1.0, P.nnz)
        P.sort_indices()
        return P

    Ps = [spread(n, mid, per_row, span // 4), spread(mid, max(2, mid // 3), 2, max(1, span // 8))]
    f = T(g.uniform(-1, 1, n))
    monkeypatch.setenv("AMGMI_POST", "fused")
    print(f"case owner form correction rows={rows} span={span} precision={precision}", flush=True)
    got = []
    for form in ("own", "pos"):
        monkeypatch.setenv("AMGMI_GALERKIN", form)
        h = AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data), precision=precision,
                smoother=rows % 2, transfer=[(T(P.indptr.astype(np.int32)), T(P.indices.astype(np.int32)), T(P.data),
                                              P.shape[1]) for P in Ps])
        z0 = h.vcycle(f)
        h.rebuild(T(1.25 * A.data))
        got.append((z0, h.vcycle(f)))
        h.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert bool(torch.isfinite(got[0][1]).all())


def test_owner_form_is_demanded(monkeypatch):
    """One row more than the form takes."""
    from paper_2108_02054_amd import AMG, AmgError
    n = 3 * 4097
    A = spd_from(n, np.arange(n - 1), np.arange(1, n), 4)
    P = sp.csr_matrix((np.ones(n), np.arange(n) // 3, np.arange(n + 1)), shape=(n, 4097))
    P2 = sp.csr_matrix((np.ones(4097), np.arange(4097) // 9, np.arange(4098)), shape=(4097, 456))
    monkeypatch.setenv("AMGMI_GALERKIN", "own")
    with pytest.raises(AmgError, match="owner form"):
        AMG(T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data),
            transfer=[(T(M.indptr.astype(np.int32)), T(M.indices.astype(np.int32)), T(M.data), M.shape[1])
                      for M in (P, P2)])
