"""3-D TV prox at the sizes where its multi-step passes can go wrong: runs of 1, 2 and 3
inner steps and their mixes, tiles of 64 depth and 24 lateral samples less a halo of the
steps on each side, runs of planes along y, batches, cold and warm starts, a modulus bound.
Against the FP64 oracle's FGP at the tolerance of the other prox tests (1e-5)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rel, to_dev, to_host

pytestmark = pytest.mark.gpu
PROX_TOL = 1e-5

CASES = [
    # (n_depth, n_x, n_y, batch), inner steps
    ((56, 18, 9, 1), 3), ((175, 36, 10, 1), 3),     # 3 steps: full lateral tiles, one depth sample past a tile
    ((60, 20, 7, 1), 2), ((120, 21, 8, 1), 4),      # 2 steps: full tiles, one row more; 4 = 2 + 2
    ((64, 45, 2, 1), 1), ((63, 21, 1, 1), 5),       # one step, one row past two tiles; a single plane
    ((120, 40, 5, 2), 10), ((6, 2, 30, 3), 7),      # batches; an image smaller than the halo
    ((126, 35, 32, 1), 11), ((16, 5, 40, 1), 30),   # more steps than the B-scan tile takes
]


@pytest.mark.parametrize("dims,inner", CASES)
@pytest.mark.parametrize("bound", [None, 0.7])
def test_tv_volume_prox(dims, inner, bound):
    import torch
    import paper_2108_01438_amd as P
    nz, nx, ny, batch = dims
    flush(f"[tv volume] {dims} inner={inner} bound={bound}")
    og, pg = both_geoms(n_depth=nz, n_x=nx, n_y=ny, n_k=nz, lateral_dims=2, batch=batch)
    plan = P.Plan(pg)
    v32, v64 = rand_image(np.random.default_rng(7), O.img_shape(og))
    vd = to_dev(v32)
    axes, tau = (3, 2, 1), 0.4
    zr, p1 = O.prox_tv(v64, tau, axes, inner, bound=bound)
    cold = plan.prox("tv", tau, 1.0, vd, tv_inner=inner, bound=bound)
    assert rel(to_host(cold), zr) <= PROX_TOL
    state = torch.zeros((3,) + O.img_shape(og), dtype=torch.complex64, device="cuda")
    warm = plan.prox("tv", tau, 1.0, vd, state=state, tv_inner=inner, bound=bound)
    assert torch.equal(torch.view_as_real(warm), torch.view_as_real(cold))   # a zero dual is a cold start
    assert rel(to_host(state), p1) <= PROX_TOL
    zr2, p2 = O.prox_tv(v64, tau, axes, inner + 1, p0=p1, bound=bound)
    z2 = plan.prox("tv", tau, 1.0, vd, state=state, tv_inner=inner + 1, bound=bound)
    assert rel(to_host(z2), zr2) <= PROX_TOL
    assert rel(to_host(state), p2) <= PROX_TOL


def test_tv_volume_prox_leaves_a_resumable_solve_alone():
    """A cold prox on the plan of an interrupted solve that left its dual in the second
    buffer takes the scratch-free route; the resumed solve still equals the whole one."""
    import torch
    import paper_2108_01438_amd as P
    og, pg = both_geoms(n_depth=64, n_x=20, n_y=12, n_k=64, lateral_dims=2)
    rng = np.random.default_rng(9)
    x32, _ = rand_image(rng, O.img_shape(og))
    plan = P.Plan(pg)
    y = plan.forward(to_dev(x32))
    delta = 1.0 / (2.1 * 64)
    whole, _ = plan.mbir_solve(y, "tv", 0.5, 7, delta=delta)
    zp = torch.empty_like(whole)
    z, _ = plan.mbir_solve(y, "tv", 0.5, 2, delta=delta, z_prev_out=zp)
    v32, v64 = rand_image(rng, O.img_shape(og))
    zc = plan.prox("tv", 0.4, 1.0, to_dev(v32), tv_inner=10)
    assert rel(to_host(zc), O.prox_tv(v64, 0.4, (3, 2, 1), 10)[0]) <= PROX_TOL
    rest, _ = plan.mbir_solve(y, "tv", 0.5, 5, delta=delta, x0=z, z_prev0=zp, k0=2)
    assert torch.equal(torch.view_as_real(rest), torch.view_as_real(whole))
