"""The marching kernels form damped Jacobi's omega / a_ii from the main diagonal they read:
the V-cycle equals the one-row-per-thread kernels' (which read the smoother's array) bit for
bit, with each smoother, each precision, symmetric and mirrored-free storage and after a
partial update; SPAI0 keeps the array."""
import gc

import numpy as np
import pytest

from tests.gpu_util import T
from workloads import two_fluid_7pt

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


@pytest.mark.parametrize("opts", [dict(), dict(smoother=1), dict(jacobi_omega=0.6), dict(npre=2, npost=2),
                                  dict(precision=1), dict(precision=1, smoother=1)])
@pytest.mark.parametrize("sym", [True, False])
def test_march_diagonal(monkeypatch, opts, sym):
    from paper_2108_02054_amd import AMG

    p, c, v0 = two_fluid_7pt(21, 0.4, ny=19, nz=13)
    v1 = two_fluid_7pt(21, 0.47, ny=19, nz=13)[2]
    r = np.random.default_rng(17).standard_normal(len(p) - 1)
    print(f"case march diagonal {opts} sym={sym}", flush=True)
    if not sym:
        monkeypatch.setenv("AMGMI_NO_DIA_SYM", "1")

    def run():
        g = AMG(T(p), T(c), T(v0), **opts)
        z = [g.vcycle(T(r)).cpu().numpy()]
        g.rebuild(T(v1))
        z.append(g.vcycle(T(r)).cpu().numpy())
        march = g.march_plane(0)
        g.close()
        return z, march

    zm, plane = run()
    monkeypatch.setenv("AMGMI_NO_MARCH", "1")
    zr, none = run()
    assert plane == 21 * 19 and none == 0
    assert np.array_equal(zm[0], zr[0]) and np.array_equal(zm[1], zr[1])
