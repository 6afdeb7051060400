"""Lateral transforms of the wide plans (radices up to 16): every radix as the first, a middle
and the last stage, two to four stages, the compile-time lengths, ragged last tiles, real-row
pairs and the y lines of volumes; and lengths that keep the radix-8 plans.  Against the FP64
oracle at the tolerance of the other operator tests (1e-5)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rand_meas, rel, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 1e-5

N_X = [96, 112, 128, 135, 144, 150, 192, 196, 210, 225, 240, 250, 256, 280,      # two and three stages
       343, 360, 378, 750, 1000, 1024, 1120, 1260, 1344, 1960, 2048, 2400, 4096,  # three
       486, 625, 1250, 2000, 3750, 3888]                                          # four, or the radix-8 plan


@pytest.mark.parametrize("nx", N_X)
@pytest.mark.parametrize("masked", [False, True])
def test_lateral_lengths(nx, masked):
    _check(dict(n_depth=64, n_x=nx, n_k=75), masked)


@pytest.mark.parametrize("nx,ny", [(96, 10), (10, 128), (150, 112), (7, 256), (256, 16)])
@pytest.mark.parametrize("masked", [False, True])
def test_lateral_lengths_of_volumes(nx, ny, masked):
    _check(dict(n_depth=64, n_x=nx, n_y=ny, n_k=50, lateral_dims=2), masked)


def _check(kw, masked):
    import paper_2108_01438_amd as P
    flush(f"[lateral] {kw} masked={masked}")
    og, pg = both_geoms(**kw)
    rng = np.random.default_rng(5)
    lat = (og.n_y if og.lateral_dims == 2 else 1, og.n_x, og.n_k)
    mask = (rng.random(lat) < 0.5).astype(np.uint8) if masked else None
    plan = P.Plan(pg, mask)
    x32, x64 = rand_image(rng, O.img_shape(og))
    r32, r64 = rand_meas(rng, O.meas_shape(og))
    yo = O.forward(x64, og, mask)
    assert rel(to_host(plan.forward(to_dev(x32))), yo) <= TOL
    assert rel(to_host(plan.adjoint(to_dev(r32))), O.adjoint(r64, og, mask)) <= TOL
    g, _ = plan.grad(to_dev(x32), to_dev(r32))
    res = yo - (r64 if mask is None else r64 * mask)
    assert rel(to_host(g), O.adjoint(res, og, mask)) <= TOL
    # one l1 iteration from a start point: the gradient step and the fused update (B-scans)
    lam, delta = 0.01 * float(np.abs(r64).max()), 1.0 / (2.1 * og.n_depth)
    z, _ = plan.mbir_solve(to_dev(r32), "l1", lam, 2, delta=delta, x0=to_dev(x32))
    zo, _ = O.fista(r64, og, mask, O.PEN_L1, lam, delta, 2, x0=x64)
    assert rel(to_host(z), zo) <= TOL
