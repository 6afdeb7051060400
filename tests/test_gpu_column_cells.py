"""Wavenumber grids whose q = 0 coordinates k_min / dk + m sit at or beside the boundary of the
base cells (2^-13 below an integer), where rounding could put two samples into one cell: every
sample of the forward, the adjoint and the gradient against the FP64 oracle at the tolerance of
the other operator tests (1e-5)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rand_meas, rel, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 1e-5
EPS = 2.0 ** -13

GRIDS = [(512, 2560 + 8191 / 8192), (1024, 20000 + 8191 / 8192 + 1e-11), (512, 2561 - 0.5 * EPS), (512, 2561 - EPS - 2e-6),
         (512, 2561 - 2 * EPS), (512, 2560 + EPS), (2048, 9000.25), (945, 3000 - 1e-9)]


@pytest.mark.parametrize("n,t0", GRIDS, ids=lambda v: f"{v!r}")
def test_grid_fraction(n, t0):
    import paper_2108_01438_amd as P
    flush(f"[column cells] n={n} k_min/dk={t0!r}")
    dk = 1.4 / n
    og, pg = both_geoms(n_depth=n, n_x=6, n_k=n + 1, k_min=t0 * dk, k_max=(t0 + n) * dk)
    rng = np.random.default_rng(5)
    plan = P.Plan(pg)
    x32, x64 = rand_image(rng, O.img_shape(og))
    r32, r64 = rand_meas(rng, O.meas_shape(og))
    yo, ao = O.forward(x64, og, None), O.adjoint(r64, og, None)
    # what an earlier call left in the workspace must not show
    plan.forward(to_dev(100.0 * x32))
    assert rel(to_host(plan.forward(to_dev(x32))), yo) <= TOL
    assert rel(to_host(plan.adjoint(to_dev(r32))), ao) <= TOL
    g, half = plan.grad(to_dev(x32), to_dev(r32))
    res = yo - r64
    assert rel(to_host(g), O.adjoint(res, og, None)) <= TOL
    assert abs(float(half) - 0.5 * np.sum(res ** 2)) <= TOL * 0.5 * np.sum(res ** 2)
