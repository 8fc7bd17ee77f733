"""BiCGStab's products on the marching storage: the SpMV that adds its own dot products
(FP64 with smoothed aggregation) and the one without (plain aggregation, FP32 hierarchies,
whose dot products are those of the other storages bit for bit)."""
import gc

import numpy as np
import pytest

from tests.gpu_util import T, rel_fro
from workloads import rhs_uniform, two_fluid_7pt
from workloads.poisson import convdiff_7pt

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_garbage():
    """Device memory held by reference cycles of an earlier test is given back first."""
    gc.collect()
    yield
    gc.collect()


# planes of several whole segments; a ragged last segment and an odd plane; one short segment
@pytest.mark.parametrize("shape", [(32, 32, 16), (33, 17, 9), (12, 11, 10)])
@pytest.mark.parametrize("sym", [False, True])  # (symmetric values: half of the diagonals read)
@pytest.mark.parametrize("opts", [dict(), dict(smoother=1), dict(aggregation=1), dict(precision=1),
                                  dict(aggregation=1, precision=1)])
def test_bicgstab_march_products(monkeypatch, shape, sym, opts):
    from paper_2108_02054_amd import AMG

    nx, ny, nz = shape
    if sym:
        p, c, v0 = two_fluid_7pt(nx, 0.4, ny=ny, nz=nz)
        v1 = two_fluid_7pt(nx, 0.47, ny=ny, nz=nz)[2]
    else:
        p, c, v0 = convdiff_7pt(nx, 0, ny=ny, nz=nz)
        v1 = convdiff_7pt(nx, 3, ny=ny, nz=nz)[2]
    f = rhs_uniform(len(p) - 1, 6, 3)
    print(f"case bicgstab march {shape} sym={sym} {opts}", flush=True)

    def run():
        g = AMG(T(p), T(c), T(v0), coarse_enough=100, **opts)
        g.rebuild(T(v1))
        out = []
        for _ in range(2):
            u, i = g.solve_bicgstab(T(f))
            out.append((u.cpu().numpy(), i))
        assert np.array_equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]  # (fixed sums)
        plane = g.march_plane(0)
        g.close()
        return *out[0], plane

    um, im, plane = run()
    monkeypatch.setenv("AMGMI_NO_MARCH", "1")
    ur, ir, none = run()
    assert plane == nx * ny and none == 0
    assert im["converged"] and ir["converged"]
    if opts.get("aggregation") or opts.get("precision"):
        assert im == ir and np.array_equal(um, ur)
    else:
        assert abs(im["iters"] - ir["iters"]) <= 1
        assert rel_fro(um, ur) <= 1e-6
