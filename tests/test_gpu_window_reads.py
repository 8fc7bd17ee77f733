"""The windowed 27-point kernels read all stored diagonals of grids that fit in the L2 caches
and half of a symmetric operator's above: both reads, and the one-row-per-thread kernels,
give the same results bit for bit on either side of the line."""
import gc

import numpy as np
import pytest

from tests.gpu_util import T
from workloads import lognormal_27pt

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


# rows at which 27 diagonals take 28 MB: 135924 in FP64, 271849 in FP32; odd row counts (the
# last thread has one row) above and below
@pytest.mark.parametrize("N,precision", [(51, 0), (53, 0), (63, 1), (65, 1)])
def test_window_reads(monkeypatch, N, precision):
    from paper_2108_02054_amd import AMG

    p, c, v0 = lognormal_27pt(N, 0)
    v1 = lognormal_27pt(N, 2)[2]
    r = np.random.default_rng(19).standard_normal(len(p) - 1)
    print(f"case window reads {N} precision {precision}", flush=True)

    def run():
        g = AMG(T(p), T(c), T(v0), precision=precision, eps_strong=0.02)
        y = g.apply_operator(T(r)).cpu().numpy()
        g.rebuild(T(v1))
        u, i = g.solve(T(r))
        z = g.vcycle(T(r)).cpu().numpy()
        out = (y, z, u.cpu().numpy(), i["iters"], g.diagonals_read(0))
        g.close()
        return out

    a = run()
    assert a[4] == 14  # found symmetric
    monkeypatch.setenv("AMGMI_NO_DIA_SYM", "1")
    b = run()
    assert b[4] == 27
    for q in range(3):
        assert np.array_equal(a[q], b[q])
    assert a[3] == b[3]
    monkeypatch.delenv("AMGMI_NO_DIA_SYM")
    monkeypatch.setenv("AMGMI_NO_WIN", "1")
    d = run()
    assert np.array_equal(a[0], d[0]) and np.array_equal(a[1], d[1])
    assert abs(a[3] - d[3]) <= 1  # (its dot products are grouped differently)
