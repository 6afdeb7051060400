"""B-scan DT-CWT levels at the edges of their tiles: depth bands of one full
tile, one more and a short last one, lateral bands that end inside a thread's
run of outputs, bands shorter than the filters (periodic wrap more than once)
and batches; against the FP64 oracle.  The tolerance is the repository's for
the shrinkage step (FP32 filters of 8 and 12 taps over at most five levels)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rand_image, rel, to_dev, to_host

pytestmark = pytest.mark.gpu

PROX_TOL = 1e-5

CASES = [
    (dict(n_depth=8, n_x=4, n_k=16), 2),                   # last lateral band: one coefficient
    (dict(n_depth=16, n_x=8, n_k=16, batch=3), 3),
    (dict(n_depth=128, n_x=16, n_k=16), 1),                # depth band 64: one tile
    (dict(n_depth=144, n_x=48, n_k=16, batch=2), 4),       # depth bands 72, 36, 18, 9
    (dict(n_depth=64, n_x=18, n_k=16), 1),                 # lateral band 9
    (dict(n_depth=280, n_x=200, n_k=16), 3),               # bands 140, 70, 35 x 100, 50, 25
    (dict(n_depth=32, n_x=1120, n_k=16, batch=2), 5),
]


@pytest.mark.parametrize("kw,levels", CASES)
def test_prox_at_tile_edges(kw, levels):
    import paper_2108_01438_amd as P
    flush(f"[dtcwt levels] {kw} levels={levels}")
    og, pg = both_geoms(**kw)
    rng = np.random.default_rng(95)
    v32, v64 = rand_image(rng, O.img_shape(og))
    plan = P.Plan(pg)
    z = to_host(plan.prox("dtcwt", 0.3, 1.0, to_dev(v32), haar_levels=levels))
    assert rel(z, O.prox_dtcwt(v64, 0.3, (3, 2), levels)) <= PROX_TOL
    plan.close()
