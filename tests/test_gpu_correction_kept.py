"""Q_l = (I - M_l A_l) P_l is kept and formed only where a V-cycle reads it."""
import gc

import numpy as np
import pytest
import torch

from tests.dense import random_spd_graph
from tests.gpu_util import T
from workloads import two_fluid_7pt

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


def live_sizes():
    from paper_2108_02054_amd.amg import ALLOC_FN, FREE_FN
    live = {}

    def a(nbytes, stream, user):
        p = torch.cuda.caching_allocator_alloc(int(nbytes), device=0, stream=int(stream or 0))
        live[p] = int(nbytes)
        return p

    def f(ptr, nbytes, stream, user):
        del live[int(ptr)]
        torch.cuda.caching_allocator_delete(int(ptr))
    return live, (ALLOC_FN(a), FREE_FN(f))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("changed", [False, True])
def test_not_in_the_coarse_tail(precision, changed):
    """Levels of the one-workgroup tail hold A P's values once, the others twice (with Q's)."""
    from paper_2108_02054_amd import AMG
    p, c, v = two_fluid_7pt(23, 0.4)
    live, cb = live_sizes()
    print(f"case correction outside the tail precision={precision} changed={changed}", flush=True)
    g = AMG(T(p), T(c), T(v), allocator=cb, coarse_enough=20, precision=precision)
    if changed:
        g.set_pattern(T(p), T(c))
        g.rebuild(T(v), pattern_changed=True)
    torch.cuda.synchronize()
    size = 4 if precision else 8
    levels = [(g.level_storage(l)["tail"], g.dims(l)[4]) for l in range(g.num_levels - 1)]
    assert {t for t, _ in levels} == {0, 1}
    for tail, nnz in levels:
        # A P's values (in FP32 also its columns are of that size), and Q's
        assert sum(b == size * nnz for b in live.values()) == 1 + precision + (0 if tail else 1), (tail, nnz)
    f = T(np.random.default_rng(1).uniform(-1, 1, len(p) - 1))
    g.rebuild(T(1.5 * v))
    u, info = g.solve(f)
    assert info["converged"]
    g.close()


# a stencil (level 0 in diagonal storage, its CSR values formed again on demand), and a general
# matrix; plain aggregation and an FP32 hierarchy, whose BiCGStab sweeps apart
@pytest.mark.parametrize("stencil", [True, False])
@pytest.mark.parametrize("opts", [dict(aggregation=1), dict(precision=1), dict(aggregation=1, precision=1, npost=2),
                                  dict(aggregation=1, smoother=1), dict(precision=1, aggregation=1, smoother=1)])
def test_updates_between_bicgstab_solves(stencil, opts):
    """They leave Q out; the first V-cycle or CG after them forms it, and what follows is bit for
    bit that of a handle that has run no BiCGStab."""
    from paper_2108_02054_amd import AMG
    p, c, v = two_fluid_7pt(21, 0.4) if stencil else random_spd_graph(4000, 5, 3)
    n = len(p) - 1
    f = T(np.random.default_rng(2).uniform(-1, 1, n))
    print(f"case corrections between BiCGStab solves stencil={stencil} {opts}", flush=True)
    a = AMG(T(p), T(c), T(v), coarse_enough=60, **opts)
    b = AMG(T(p), T(c), T(v), coarse_enough=60, **opts)
    products = lambda: a.trace_read().get("galerkin_ap", (0, 0))[1]  # noqa: E731
    levels = a.num_levels - 1
    tails = sum(a.level_storage(l)["tail"] for l in range(levels))
    a.trace(["galerkin_ap"], level=-1)
    for step in range(1, 4):
        w = T((1.0 + 0.3 * step) * v)
        a.rebuild(T((1.0 + 0.2 * step) * v))
        products()
        _, info = a.solve_bicgstab(f)
        assert info["converged"] and products() == 0
        a.rebuild(w)
        b.rebuild(w)
        assert products() == levels
        if step == 2:  # straight to CG
            ua, ia = a.solve(f)
            assert products() == levels - tails
            ub, ib = b.solve(f)
            assert ia == ib and torch.equal(ua, ub)
        else:
            assert torch.equal(a.vcycle(f), b.vcycle(f))
            assert products() == levels - tails
        assert torch.equal(a.vcycle(f), b.vcycle(f)) and products() == 0
        w = T((1.0 + 0.4 * step) * v)  # an update after such a cycle brings Q itself
        a.rebuild(w)
        b.rebuild(w)
        assert torch.equal(a.vcycle(f), b.vcycle(f)) and products() == levels
        a.solve_bicgstab(f)  # both kinds of solve on the same values: the update brings Q
        a.rebuild(w)
        assert torch.equal(a.vcycle(f), b.vcycle(f)) and products() == levels
    a.close()
    b.close()


def budget(limit):
    """The caller's allocator with at most `limit` bytes out at a time; the most that were."""
    from paper_2108_02054_amd.amg import ALLOC_FN, FREE_FN
    st = dict(live=0, peak=0, refused=0)

    def a(nbytes, stream, user):
        if st["live"] + nbytes > limit:
            st["refused"] += 1
            return None
        st["live"] += nbytes
        st["peak"] = max(st["peak"], st["live"])
        return torch.cuda.caching_allocator_alloc(int(nbytes), device=0, stream=int(stream or 0))

    def f(ptr, nbytes, stream, user):
        st["live"] -= nbytes
        torch.cuda.caching_allocator_delete(int(ptr))
    return st, (ALLOC_FN(a), FREE_FN(f))


@pytest.mark.parametrize("kind,opts", [
    ("stencil", dict()), ("stencil", dict(aggregation=1)), ("stencil", dict(precision=1, aggregation=1)),
    ("graph", dict()), ("graph", dict(precision=1))])
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("bicgstab", [False, True])
def test_not_refused_for_its_memory(monkeypatch, kind, opts, bicgstab, full):
    """A series that fits in the memory of a hierarchy without Q is set up, updated and solved in
    that memory, by a first setup and by a full rebuild."""
    from paper_2108_02054_amd import AMG, FULL
    p, c, v = two_fluid_7pt(40, 0.4) if kind == "stencil" else random_spd_graph(8000, 5, 3)
    f = T(np.random.default_rng(4).uniform(-1, 1, len(p) - 1))
    print(f"case memory without corrections {kind} {opts} bicgstab={bicgstab} full={full}", flush=True)

    def series(limit):
        st, cb = budget(limit)
        g = AMG(T(p), T(c), T(v), allocator=cb, coarse_enough=200, **opts)
        solve = lambda: (g.solve_bicgstab(f) if bicgstab else g.solve(f))[1]  # noqa: E731
        g.rebuild(T(1.5 * v))
        one = solve()
        if full:
            g.rebuild_ex(T(v), FULL)
        two = solve()
        assert bool(torch.isfinite(g.vcycle(f)).all())
        g.close()
        assert st["live"] == 0
        return st, one, two

    monkeypatch.setenv("AMGMI_POST", "sweep")
    lean, one, two = series(1 << 40)
    monkeypatch.delenv("AMGMI_POST")
    wide = series(1 << 40)[0]
    got, a, b = series(lean["peak"])
    assert got["peak"] <= lean["peak"] and (got["refused"] > 0) == (wide["peak"] > lean["peak"])
    assert full or got["refused"] > 0
    for x, y in ((a, one), (b, two)):
        assert x["converged"] and abs(x["iters"] - y["iters"]) <= (4 if bicgstab else 1)
