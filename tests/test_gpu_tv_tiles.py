"""B-scan TV prox at the edges of its tiles (64 depth samples by 72 or 128 lateral ones, less
a halo of the inner steps on each side): one full tile, one sample more, both tile widths,
the most steps a tile takes and one more, batches, cold and warm starts, a modulus bound;
and the objective's TV value, whose tiles are one sample smaller.  Against the FP64 oracle's
FGP at the tolerance of the other prox tests (1e-5)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rel, to_dev, to_host

pytestmark = pytest.mark.gpu
PROX_TOL = 1e-5

CASES = [
    # (n_depth, n_x, batch), inner steps
    ((42, 50, 1), 10), ((45, 54, 1), 10), ((84, 105, 2), 10), ((90, 100, 1), 10),   # cores 43 x 51
    ((60, 70, 1), 1), ((63, 72, 3), 1), ((125, 140, 1), 1),                         # cores 61 x 69
    ((30, 90, 1), 16), ((32, 98, 1), 16), ((64, 192, 2), 16),   # cores 31 x 95 of the wide tile
    ((9, 72, 1), 27), ((28, 150, 1), 27), ((28, 40, 1), 28),    # most steps of a tile, and one more
    ((6, 2, 4), 10), ((8, 1000, 1), 12),                        # smaller than the halo; one tile deep
]


@pytest.mark.parametrize("dims,inner", CASES)
@pytest.mark.parametrize("bound", [None, 0.7])
def test_tv_bscan_tiles(dims, inner, bound):
    import torch
    import paper_2108_01438_amd as P
    nz, nx, batch = dims
    flush(f"[tv tiles] {dims} inner={inner} bound={bound}")
    og, pg = both_geoms(n_depth=nz, n_x=nx, n_k=max(nz, 16), batch=batch)
    plan = P.Plan(pg)
    v32, v64 = rand_image(np.random.default_rng(8), O.img_shape(og))
    vd = to_dev(v32)
    axes, tau = (3, 2), 0.4
    zr, p1 = O.prox_tv(v64, tau, axes, inner, bound=bound)
    cold = plan.prox("tv", tau, 1.0, vd, tv_inner=inner, bound=bound)
    assert rel(to_host(cold), zr) <= PROX_TOL
    state = torch.zeros((2,) + O.img_shape(og), dtype=torch.complex64, device="cuda")
    plan.prox("tv", tau, 1.0, vd, state=state, tv_inner=inner, bound=bound)
    assert rel(to_host(state), p1) <= PROX_TOL
    zr2, p2 = O.prox_tv(v64, tau, axes, 7, p0=p1, bound=bound)
    z2 = plan.prox("tv", tau, 1.0, vd, state=state, tv_inner=7, bound=bound)
    assert rel(to_host(z2), zr2) <= PROX_TOL
    assert rel(to_host(state), p2) <= PROX_TOL
    plan.close()


@pytest.mark.parametrize("dims,inner", [((42, 48, 1), 10), ((90, 108, 2), 10), ((64, 192, 1), 16)])
def test_tv_objective_uses_its_own_tiles(dims, inner):
    import paper_2108_01438_amd as P
    nz, nx, batch = dims
    og, pg = both_geoms(n_depth=nz, n_x=nx, n_k=nz, batch=batch)
    plan = P.Plan(pg)
    x32, _ = rand_image(np.random.default_rng(10), O.img_shape(og))
    y = plan.forward(to_dev(x32))
    y64 = to_host(y).astype(np.float64)
    delta, lam = 1.0 / (2.1 * nz), 0.5
    zo, ho = O.fista(y64, og, None, O.PEN_TV, lam, delta, 6, tv_inner=inner)
    z, info = plan.mbir_solve(y, "tv", lam, 6, delta=delta, tv_inner=inner, objective=True)
    assert rel(to_host(z), zo) <= 1e-4                       # the solver tests' tolerances
    np.testing.assert_allclose(info["objective"], ho, rtol=1e-5)
    z2, _ = plan.mbir_solve(y, "tv", lam, 6, delta=delta, tv_inner=inner)
    assert np.array_equal(to_host(z2), to_host(z))
    plan.close()
