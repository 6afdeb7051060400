"""Column pairs on the twice oversampled grid: transform plans of two to four stages and the
compile-time lengths, few and many pairs (two and five base cells per thread), windows of 4,
6 and 8 taps, empty base cells, evanescent samples, columns whose samples drift across a cell
boundary, and the geometries next to the rule's limits that take the general kernels.
Against the FP64 oracle at the tolerance of the other operator tests (1e-5)."""
import math

import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rand_meas, rel, to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 1e-5
DZ0 = 0.5 * math.pi / (2.0 * math.pi / 0.75 - 2.0 * math.pi / 0.9)   # n_depth dz / (n_k - 1) of the default pitch

CASES = [
    # two stages, three (the smallest radices too), four; odd lengths
    dict(n_depth=64, n_x=7, n_k=96), dict(n_depth=126, n_x=5, n_k=101), dict(n_depth=125, n_x=6, n_k=125),
    dict(n_depth=945, n_x=3, n_k=1003), dict(n_depth=1225, n_x=4, n_k=1100), dict(n_depth=1400, n_x=5, n_k=1400),
    dict(n_depth=2016, n_x=3, n_k=1800), dict(n_depth=2025, n_x=2, n_k=2300),
    # no plan: the general kernels
    dict(n_depth=60, n_x=6, n_k=70), dict(n_depth=2000, n_x=3, n_k=1500),
    # compile-time lengths with few pairs; many pairs (five cells per thread)
    dict(n_depth=512, n_x=9, n_k=520), dict(n_depth=1024, n_x=6, n_k=900), dict(n_depth=2048, n_x=4, n_k=2048),
    dict(n_depth=512, n_x=540, n_k=500), dict(n_depth=1024, n_x=525, n_k=1024), dict(n_depth=80, n_x=525, n_k=90),
    dict(n_depth=72, n_x=20, n_y=30, n_k=75, lateral_dims=2),
    # tap counts
    dict(n_depth=96, n_x=600, n_k=110, kb_width=4), dict(n_depth=96, n_x=8, n_k=110, kb_width=8),
    dict(n_depth=128, n_x=7, n_k=64, kb_width=8, batch=3),
    # sample spacings: 1.5 cells (empty cells), past the grid and below a cell (general kernels)
    dict(n_depth=128, n_x=9, n_k=100, dz=1.5 * DZ0 * 99 / 128), dict(n_depth=128, n_x=9, n_k=200, dz=2.0 * DZ0 * 199 / 128),
    dict(n_depth=128, n_x=9, n_k=100, dz=0.7 * DZ0 * 99 / 128),
    # evanescent samples in the outer columns; every sample of some columns evanescent
    dict(n_depth=64, n_x=24, n_k=64, k_min=0.3, k_max=0.9, dx=0.9), dict(n_depth=80, n_x=525, n_k=64, k_min=0.3, k_max=0.9, dx=0.9),
    dict(n_depth=80, n_x=25, n_k=64, k_min=0.3, k_max=0.9, dx=0.5),
    # a focus off the middle (its phase per sample)
    dict(n_depth=160, n_x=10, n_k=150, z_focus=12.0, disp_b=1e-6),
]


def _drift(factor):
    """A geometry whose first off-axis column has t_m = integer - factor 2^-13 in mid-band."""
    n_k, n_x = 300, 6
    ct = 0.5 * (n_k - 1) / (2.0 * math.pi / 0.75 - 2.0 * math.pi / 0.9)
    q = math.sqrt(factor * 2.0 ** -13 * 4.0 * 7.68 / ct)
    return dict(n_depth=256, n_x=n_x, n_k=n_k, dx=2.0 * math.pi / (n_x * q))


CASES += [_drift(f) for f in (0.9, 1.0, 1.1)]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join(f"{k}{v:.4g}" for k, v in kw.items()))
@pytest.mark.parametrize("masked", [False, True])
def test_columns(kw, masked):
    import paper_2108_01438_amd as P
    flush(f"[columns] {kw} masked={masked}")
    og, pg = both_geoms(**kw)
    rng = np.random.default_rng(21)
    lat = (og.n_y if og.lateral_dims == 2 else 1, og.n_x, og.n_k)
    mask = (rng.random(lat) < 0.5).astype(np.uint8) if masked else None
    plan = P.Plan(pg, mask)
    x32, x64 = rand_image(rng, O.img_shape(og))
    r32, r64 = rand_meas(rng, O.meas_shape(og))
    yo, ao = O.forward(x64, og, mask), O.adjoint(r64, og, mask)
    assert rel(to_host(plan.forward(to_dev(x32))), yo) <= TOL
    assert rel(to_host(plan.adjoint(to_dev(r32))), ao) <= TOL
    g, half = plan.grad(to_dev(x32), to_dev(r32))
    res = yo - (r64 if mask is None else r64 * mask)
    assert rel(to_host(g), O.adjoint(res, og, mask)) <= TOL
    assert abs(float(half) - 0.5 * np.sum(res ** 2)) <= TOL * 0.5 * np.sum(res ** 2)
