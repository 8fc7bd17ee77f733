"""The coarse correction and the first post-sweep in one pass (Q = (I - M A) P on A P's
pattern) against the separate prolongation and sweep, and against the oracle's V-cycle."""
import gc

import numpy as np
import pytest

from tests.gpu_util import T, both, rel_max
from workloads import lognormal_27pt, two_fluid_7pt

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


def problem(kind):
    if kind == "7pt":
        return two_fluid_7pt(23, 0.4, ny=17, nz=19), two_fluid_7pt(23, 0.55, ny=17, nz=19)[2]
    if kind == "27pt":
        p, c, v = lognormal_27pt(14, 0)
        return (p, c, v), lognormal_27pt(14, 3)[2]
    # a graph with rows of 1 to 40 entries (general CSR on level 0), strictly dominant
    g = np.random.default_rng(5)
    n = 1500
    i = np.concatenate([np.arange(n - 1), g.integers(0, n, 2 * n), np.zeros(30, int)])
    j = np.concatenate([np.arange(1, n), g.integers(0, n, 2 * n), g.integers(1, n, 30)])
    A = np.zeros((n, n))
    w = -g.uniform(0.1, 1.0, i.size)
    A[i, j] += w
    A[j, i] += w
    np.fill_diagonal(A, 0.0)
    A[np.arange(n), np.arange(n)] = 0.01 - A.sum(axis=1)
    rows, cols = np.nonzero(A)
    p = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    return (p, cols.astype(np.int32), A[rows, cols]), 1.5 * A[rows, cols]


@pytest.mark.parametrize("kind", ["7pt", "27pt", "graph"])
@pytest.mark.parametrize("opts", [dict(), dict(smoother=1), dict(aggregation=1), dict(npost=2), dict(npre=0),
                                  dict(npre=2), dict(precision=1), dict(precision=1, aggregation=1),
                                  dict(flexible_cg=1)])
def test_fused_correction(monkeypatch, kind, opts):
    (p, c, v0), v1 = problem(kind)
    n = len(p) - 1
    opts = dict(coarse_enough=40, **opts)
    f = np.random.default_rng(3).uniform(-1, 1, n)
    print(f"case fused correction {kind} {opts}", flush=True)
    monkeypatch.setenv("AMGMI_POST", "fused")
    g, o = both(p, c, v0, **opts)
    monkeypatch.setenv("AMGMI_POST", "sweep")
    h, _ = both(p, c, v0, **opts)
    # FP64: the two forms and the oracle differ by rounding, a few eps per level times the
    # operator's condition within a sweep; FP32 the same in its own eps
    tol = 1e-10 if opts.get("precision", 0) == 0 else 2e-4
    for step in range(2):  # as set up, and after a partial update
        if step:
            g.rebuild(T(v1))
            h.rebuild(T(v1))
            o.rebuild(v1, 0)
        zg, zh, zo = g.vcycle(T(f)).cpu().numpy(), h.vcycle(T(f)).cpu().numpy(), o.vcycle(f)
        assert rel_max(zg, zh) <= tol and rel_max(zg, zo) <= tol
        ug, ig = g.solve(T(f))
        uh, ih = h.solve(T(f))
        assert ig["converged"] == ih["converged"] and abs(ig["iters"] - ih["iters"]) <= 1
        if ig["converged"]:
            assert rel_max(ug.cpu().numpy(), uh.cpu().numpy()) <= 1e-6
    g.close()
    h.close()
