"""Block systems: the restriction with the next level's first sweep, the first post-sweep
with the coarse correction, and the CG update with level 0's first sweep, against the
oracle and against the cycle with a prolongation pass of its own."""
import gc

import numpy as np
import pytest
import scipy.sparse as sp

from tests.dense import random_spd_graph
from tests.gpu_util import T, both, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


def system(bs, isolated):
    pp, cc, vv = random_spd_graph(1100, 5, bs)
    rg = np.random.default_rng(bs)
    M = rg.uniform(-1.0, 1.0, size=(bs, bs))
    N = sp.csr_matrix((vv, cc, pp), shape=(1100, 1100))
    if isolated:  # nodes outside every aggregate: the correction adds nothing to them
        N = sp.block_diag([N, sp.identity(37) * N.diagonal().max()], format="csr")
    A = sp.kron(N, sp.csr_matrix(M @ M.T + bs * np.eye(bs)), format="csr")
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.copy()


# 2, 4, 8: all three fused; 3, 6: the correction only (row blocks and wavefronts would cut nodes)
@pytest.mark.parametrize("bs", [2, 3, 4, 6, 8])
@pytest.mark.parametrize("opts", [dict(), dict(npost=2), dict(npre=2), dict(npre=0), dict(npost=0),
                                  dict(precision=1)])
@pytest.mark.parametrize("isolated", [False, True])
def test_block_cycle_fused(monkeypatch, bs, opts, isolated):
    p, c, v = system(bs, isolated)
    n = len(p) - 1
    prm = dict(block_size=bs, aggregation=1, coarse_enough=12 * bs, **opts)
    print(f"case block cycle bs={bs} {opts} isolated={isolated}", flush=True)
    f = np.random.default_rng(7).uniform(-1.0, 1.0, n)
    g, o = both(p, c, v, **prm)
    assert g.num_levels >= 3
    monkeypatch.setenv("AMGMI_NO_NODE_TRANSFER", "1")
    h, _ = both(p, c, v, **prm)
    # a few eps per level times the conditioning within a sweep, in the cycle's precision
    tol = 1e-10 if opts.get("precision", 0) == 0 else 2e-4
    for step in range(2):  # as set up, and after a partial update
        if step:
            g.rebuild(T(1.7 * v))
            h.rebuild(T(1.7 * v))
            o.rebuild(1.7 * v, 0)
        zg, zh = g.vcycle(T(f)).cpu().numpy(), h.vcycle(T(f)).cpu().numpy()
        assert np.array_equal(zg, zh)  # the sum u + P uc is the one a pass of its own stores
        assert rel_max(zg, o.vcycle(f)) <= tol
        ug, ig = g.solve(T(f))
        uh, ih = h.solve(T(f))
        assert ig == ih and np.array_equal(ug.cpu().numpy(), uh.cpu().numpy())
        if opts.get("npre", 1) == opts.get("npost", 1):  # (a symmetric cycle)
            assert ig["converged"]
            A = sp.csr_matrix(((1.7 if step else 1.0) * v, c, p), shape=(n, n))
            assert np.linalg.norm(f - A @ ug.cpu().numpy()) <= 2e-8 * np.linalg.norm(f)
    g.close()
    h.close()


# the sweep that a restriction (levels below 0) and a CG update (level 0) form, and the pass
# that forms it where they cannot, add the same products in the same order, each rounded
@pytest.mark.parametrize("bs", [2, 4, 8])
@pytest.mark.parametrize("precision", [0, 1])
def test_first_sweeps_bit_for_bit(monkeypatch, bs, precision):
    from paper_2108_02054_amd import AMG
    p, c, v = system(bs, True)
    n = len(p) - 1
    f = np.random.default_rng(8).uniform(-1.0, 1.0, n)
    print(f"case first sweeps bs={bs} precision={precision}", flush=True)
    got = []
    for apart in (False, True):
        if apart:
            monkeypatch.setenv("AMGMI_NO_NODE_SWEEPS", "1")
        g = AMG(T(p), T(c), T(v), block_size=bs, aggregation=1, coarse_enough=12 * bs, precision=precision)
        assert g.num_levels >= 3
        z = g.vcycle(T(f)).cpu().numpy()
        u, i = g.solve(T(f))
        got.append((z, u.cpu().numpy(), i))
        g.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert got[0][2] == got[1][2] and np.array_equal(got[0][1], got[1][1])
