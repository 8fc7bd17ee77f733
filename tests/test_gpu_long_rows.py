"""Setup of matrices with a few rows far longer than the rest (hubs): patterns and values as
the oracle's at the lengths where the row kernels change form, and no time that grows with
the square of the length."""
import gc
import time

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from tests.gpu_util import T, both, compare_levels

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


def laplacian(n, i, j, w):
    W = sp.coo_matrix((-np.asarray(w, float), (i, j)), shape=(n, n))
    W = (W + W.T).tocsr()
    W.setdiag(0)
    W.eliminate_zeros()
    A = (W + sp.diags(1.0 - np.asarray(W.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return A


def band_with_hub(n, width, links, strong, seed):
    """A band graph of `width` neighbours to each side; node n // 2 has weak links to `links`
    more nodes and strong ones to `strong` of those."""
    g = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), width)
    j = np.minimum(i + np.tile(np.arange(1, width + 1), n), n - 1)
    h = n // 2
    far = np.setdiff1d(np.arange(n), np.arange(h - width, h + width + 1))
    to = g.choice(far, links, replace=False)
    w = np.full(links, 1e-5)
    w[:strong] = 2.0
    return laplacian(n, np.r_[i, np.full(links, h)], np.r_[j, to], np.r_[g.uniform(0.5, 1.5, len(i)), w])


# rows of 5, 9, 19 and 45 entries take 4, 8, 16 and 32 lanes; the hub's row has 16 entries per
# lane, one more, and far more
@pytest.mark.parametrize("width,lanes", [(2, 4), (4, 8), (9, 16), (22, 32)])
@pytest.mark.parametrize("extra", [0, 1, 777])
def test_hub_rows_as_oracle(width, lanes, extra):
    n = 2600
    A = band_with_hub(n, width, 16 * lanes + extra - 2 * width - 1, 7, 11 + width)
    length = int(np.diff(A.indptr).max())
    assert length == 16 * lanes + extra
    print(f"case hub row of {length} entries, {lanes} lanes", flush=True)
    g, o = both(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, coarse_enough=20, eps_strong=0.02)
    hub = g.level(0)["P"]
    assert hub[0][n // 2 + 1] - hub[0][n // 2] >= 3  # several aggregates
    compare_levels(g, o, tol=1e-12)
    g.close()


def test_star_setup_time():
    """A star of 8000 nodes: every entry of its long row is strong.  (About 20 ms; 2.3 s with a
    comparison of all pairs of entries.)"""
    from paper_2108_02054_amd import AMG
    n = 8000
    A = laplacian(n, np.zeros(n - 1, int), np.arange(1, n), np.random.default_rng(1).uniform(0.1, 1.0, n - 1))
    p, c, v = T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data)
    took = []
    for _ in range(3):
        torch.cuda.synchronize()
        t = time.perf_counter()
        g = AMG(p, c, v, eps_strong=1e-3)
        torch.cuda.synchronize()
        took.append(time.perf_counter() - t)
        g.close()
    print(f"case star of {n} nodes: {1e3 * min(took):.1f} ms", flush=True)
    assert min(took) < 0.4


@pytest.mark.parametrize("n", [6000, 9000])
def test_hub_product_pattern_time(n):
    """A chain whose nodes all have a weak link to one: the hub's rows of the Galerkin products
    overflow the tables of the short rows.  (6000 nodes: symbolic phase about 9 ms; 80 ms with
    every term probing a full table.)"""
    from paper_2108_02054_amd import AMG
    g = np.random.default_rng(2)
    i = np.r_[np.arange(n - 1), np.zeros(n - 2, int)]
    j = np.r_[np.arange(1, n), np.arange(2, n)]
    A = laplacian(n, i, j, np.r_[g.uniform(0.5, 1.5, n - 1), np.full(n - 2, 1e-6)])
    p, c, v = T(A.indptr.astype(np.int32)), T(A.indices.astype(np.int32)), T(A.data)
    took = []
    for _ in range(3):
        h = AMG(p, c, v, aggregation=1)
        took.append(h.phase_times()["symbolic"])
        h.close()
    print(f"case hub product of {n} nodes: symbolic {min(took):.1f} ms", flush=True)
    assert min(took) < 40.0
