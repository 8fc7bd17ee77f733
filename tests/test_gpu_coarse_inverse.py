"""The dense inverse of the coarsest operator at the edges of its tiles: 16-pivot blocks in
one workgroup up to 128 rows, 64-pivot blocks over the device above (an odd or an even
number of block steps, a ragged last block)."""
import gc

import numpy as np
import pytest

from tests.gpu_util import T, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


def band_spd(n, seed):
    """A symmetric, strictly diagonally dominant matrix: 12 random couplings per row at most,
    condition number below 40."""
    g = np.random.default_rng(seed)
    A = np.zeros((n, n))
    for d in (1, 2, 7, 16, 33, 64):
        if d < n:
            w = -g.uniform(0.1, 1.0, n - d)
            A += np.diag(w, d) + np.diag(w, -d)
    A += np.diag(1.0 - A.sum(axis=1))
    return A


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 32, 63, 65, 112, 127, 128, 129, 192, 193, 257, 400])
@pytest.mark.parametrize("precision", [0, 1])
def test_inverse_sizes(n, precision):
    from paper_2108_02054_amd import AMG
    A = band_spd(n, n)
    rows, cols = np.nonzero(A)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    val = A[rows, cols]
    print(f"case coarse inverse n={n} precision {precision}", flush=True)
    g = AMG(T(ptr), T(cols.astype(np.int32)), T(val), coarse_enough=2048, precision=precision)
    assert g.num_levels == 1
    for scale in (1.0, 3.0):  # as set up, and after a partial update
        if scale != 1.0:
            g.rebuild(T(scale * val))
        B = A if precision == 0 else A.astype(np.float32).astype(np.float64)
        if scale != 1.0:
            B = scale * A if precision == 0 else (scale * A).astype(np.float32).astype(np.float64)
        # elimination error: about n cond eps < 400 * 40 * 1.2e-16 = 2e-12
        assert rel_max(g.coarse_inverse(), np.linalg.inv(B)) <= 4e-12
    g.close()


@pytest.mark.parametrize("n", [40, 200])
def test_negative_pivot_is_reported(n):
    """A late pivot that is not positive, in one workgroup and in a later 64-pivot block."""
    from paper_2108_02054_amd import AMG, AmgError
    A = band_spd(n, 1)
    A[n - 1, n - 2] = A[n - 2, n - 1] = -40.0
    rows, cols = np.nonzero(A)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    print(f"case negative pivot n={n}", flush=True)
    with pytest.raises(AmgError, match="NOT_SPD"):
        AMG(T(ptr), T(cols.astype(np.int32)), T(A[rows, cols]), coarse_enough=2048)
