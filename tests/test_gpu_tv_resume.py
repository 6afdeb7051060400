"""A TV solve interrupted after an even or an odd number of iterations (its dual then sits in
the plan's second or first buffer), TV prox calls on the same plan, and the rest of the solve:
the two parts equal the whole solve bitwise, and the prox calls the oracle (1e-5, as the other
TV prox tests)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rel, to_dev, to_host

pytestmark = pytest.mark.gpu
PROX_TOL = 1e-5


@pytest.mark.parametrize("kw", [dict(n_depth=96, n_x=40, n_k=90), dict(n_depth=64, n_x=20, n_y=12, n_k=64, lateral_dims=2)],
                         ids=["bscan", "volume"])
@pytest.mark.parametrize("first", [2, 3])
@pytest.mark.parametrize("inner", [3, 10])
@pytest.mark.parametrize("with_state", [False, True])
def test_prox_between_the_parts_of_a_solve(kw, first, inner, with_state):
    import torch
    import paper_2108_01438_amd as P
    flush(f"[tv resume] {kw} first={first} inner={inner} state={with_state}")
    og, pg = both_geoms(**kw)
    axes = (3, 2, 1) if og.lateral_dims == 2 else (3, 2)
    rng = np.random.default_rng(9)
    x32, _ = rand_image(rng, O.img_shape(og))
    plan = P.Plan(pg)
    y = plan.forward(to_dev(x32))
    delta = 1.0 / (2.1 * og.n_depth)
    whole, _ = plan.mbir_solve(y, "tv", 0.5, 7, delta=delta)
    zp = torch.empty_like(whole)
    z, _ = plan.mbir_solve(y, "tv", 0.5, first, delta=delta, z_prev_out=zp)
    v32, v64 = rand_image(rng, O.img_shape(og))
    state = torch.zeros((og.lateral_dims + 1,) + O.img_shape(og), dtype=torch.complex64, device="cuda") if with_state else None
    zc = plan.prox("tv", 0.4, 1.0, to_dev(v32), state=state, tv_inner=inner)
    zr, pr = O.prox_tv(v64, 0.4, axes, inner)
    assert rel(to_host(zc), zr) <= PROX_TOL
    if with_state:
        assert rel(to_host(state), pr) <= PROX_TOL
    rest, _ = plan.mbir_solve(y, "tv", 0.5, 7 - first, delta=delta, x0=z, z_prev0=zp, k0=first)
    assert torch.equal(torch.view_as_real(rest), torch.view_as_real(whole))
