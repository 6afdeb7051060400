"""Wide lateral plans at run-time lengths on launches large enough for them (the small images of
test_gpu_lateral_plans.py with one stage less keep the radix-8 plans): tiles of one to sixteen rows,
one to three stages saved, a ragged last tile, and lengths on either side of the rule: two-row tiles
with one stage less, and one-row tiles that the wide plan widens, few and many.  Against the FP64
oracle at the tolerance of that file (1e-5)."""
import pytest

import test_gpu_lateral_plans as base

pytestmark = pytest.mark.gpu

CASES = [
    dict(n_depth=35, n_x=280, n_k=36, batch=30), dict(n_depth=32, n_x=600, n_k=30, batch=24),   # one stage less
    dict(n_depth=16, n_x=1120, n_k=17, batch=33), dict(n_depth=40, n_x=1600, n_k=40, batch=13),
    dict(n_depth=32, n_x=1400, n_k=32, batch=16), dict(n_depth=16, n_x=4000, n_k=16, batch=17),
    dict(n_depth=35, n_x=810, n_k=40, batch=8), dict(n_depth=21, n_x=1250, n_k=24, batch=6),    # two and three less
    dict(n_depth=40, n_x=2240, n_k=32, batch=1), dict(n_depth=12, n_x=2560, n_k=12, batch=3),   # two rows, one stage less
    dict(n_depth=48, n_x=2058, n_k=48, batch=6), dict(n_depth=16, n_x=3840, n_k=18, batch=1),   # one row to two
    dict(n_depth=64, n_x=70, n_y=24, n_k=50, lateral_dims=2), dict(n_depth=16, n_x=24, n_y=600, n_k=18, lateral_dims=2),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
@pytest.mark.parametrize("masked", [False, True])
def test_wide_plans(kw, masked):
    base._check(dict(kw), masked)
