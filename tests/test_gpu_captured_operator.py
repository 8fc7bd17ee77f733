"""The operator captured into a graph multiplies by the values of the latest partial update:
a system that is symmetric when the graph is captured (a flow at rest) need not be so at a
replay."""
import ctypes as C
import gc

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from tests.gpu_util import T
from workloads import lognormal_27pt, two_fluid_7pt

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


# the marching kernels (7-point) and the windowed ones on both sides of the size from which
# they read half of a symmetric operator (27-point)
@pytest.mark.parametrize("points,N", [(7, 24), (27, 12), (27, 51), (27, 53)])
@pytest.mark.parametrize("after_solve", [False, True])
def test_captured_operator_follows_unsymmetric_values(points, N, after_solve):
    from paper_2108_02054_amd import AMG, lib
    p, c, v = two_fluid_7pt(N, 0.4) if points == 7 else lognormal_27pt(N, 0)
    n = len(p) - 1
    g = np.random.default_rng(N)
    x = g.uniform(-1, 1, n)
    print(f"case captured operator {points} points {N}^3 after_solve={after_solve}", flush=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        h = AMG(T(p), T(c), T(v), eps_strong=0.08 if points == 7 else 0.02)
        X, Y = T(x), torch.empty(n, dtype=torch.float64, device="cuda")
        if after_solve:
            h.solve(X)
        call = lambda: lib().amg_apply_operator_noalloc(h.ctx, C.c_void_p(X.data_ptr()), C.c_void_p(Y.data_ptr()))  # noqa: E731
        assert call() == 0
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            assert call() == 0
        for step in range(3):
            w = v if step == 0 else v * g.uniform(0.5, 1.5, len(v))  # unsymmetric from step 1 on
            h.rebuild(T(w))
            Y.fill_(float("nan"))
            graph.replay()
            side.synchronize()
            got = Y.cpu().numpy()
            eager = h.apply_operator(X)
            side.synchronize()
            A = sp.csr_matrix((w, c, p), shape=(n, n))
            # a row adds at most 27 rounded products
            assert np.abs(got - A @ x).max() <= 30 * 2.3e-16 * (abs(A) @ abs(x)).max()
            assert np.array_equal(got, eager.cpu().numpy())
        del graph
        h.close()
    torch.cuda.current_stream().wait_stream(side)


# a hierarchy whose every pass runs on the context's own stream (a coarsest level of at most 128
# rows): its V-cycle can be captured as well
@pytest.mark.parametrize("opts", [dict(), dict(aggregation=1), dict(precision=1), dict(smoother=1)])
@pytest.mark.parametrize("after_solve", [False, True])
def test_captured_cycle_follows_updates(opts, after_solve):
    from paper_2108_02054_amd import AMG
    p, c, v = two_fluid_7pt(22, 0.4)
    n = len(p) - 1
    g = np.random.default_rng(3)
    f = g.uniform(-1, 1, n)
    print(f"case captured cycle {opts} after_solve={after_solve}", flush=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        h = AMG(T(p), T(c), T(v), coarse_enough=60, **opts)
        F = T(f)
        if after_solve:
            h.solve(F)
        h.vcycle(F)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            Z = h.vcycle(F)
        for step in range(4):
            # step 1: unsymmetric values; then solves that read no Q between the updates
            w = v if step == 0 else v * (1.0 + 0.02 * g.uniform(-1, 1, len(v)))
            h.rebuild(T(w))
            if step >= 2:
                h.solve_bicgstab(F)
                w = 1.5 * w
                h.rebuild(T(w))
            graph.replay()
            side.synchronize()
            got = Z.cpu().numpy()
            want = h.vcycle(F)
            side.synchronize()
            assert np.array_equal(got, want.cpu().numpy()), step
        del graph
        h.close()
    torch.cuda.current_stream().wait_stream(side)


@pytest.mark.parametrize("opts", [dict(aggregation=1), dict(precision=1)])
def test_cycle_captured_where_an_update_left_q_out(opts):
    """The forming of Q is recorded with the cycle; an eager cycle still forms its own."""
    from paper_2108_02054_amd import AMG
    p, c, v = two_fluid_7pt(22, 0.4)
    f = np.random.default_rng(3).uniform(-1, 1, len(p) - 1)
    print(f"case captured cycle that forms Q {opts}", flush=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        h, o = (AMG(T(p), T(c), T(v), coarse_enough=60, **opts) for _ in range(2))
        F = T(f)
        h.vcycle(F)  # (every kernel of the cycle has run once before the capture)
        h.rebuild(T(1.1 * v))
        h.solve_bicgstab(F)
        for x in (h, o):
            x.rebuild(T(1.4 * v))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            Z = h.vcycle(F)
        want = o.vcycle(F)
        assert torch.equal(h.vcycle(F), want)
        graph.replay()
        assert torch.equal(Z, want)
        assert np.array_equal(h.level(0)["A"][2], o.level(0)["A"][2])
        for x in (h, o):
            x.rebuild(T(1.7 * v))
        graph.replay()
        assert torch.equal(Z, o.vcycle(F)) and torch.equal(h.vcycle(F), o.vcycle(F))
        assert np.array_equal(h.level(0)["A"][2], o.level(0)["A"][2])
        side.synchronize()
        del graph
        h.close()
        o.close()
    torch.cuda.current_stream().wait_stream(side)
