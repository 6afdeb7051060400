"""B-scan TV prox at sizes that take the 64 x 128 tiles (the 64 x 72 ones just miss a round of
workgroups there; small images take the latter): ten, 16 and 22 steps, one sample past full tiles,
batches; and the objective's TV value on them.  Against the FP64 oracle at the tolerance of
test_gpu_tv_tiles.py (1e-5)."""
import pytest

import test_gpu_tv_tiles as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,inner", [((600, 1890, 1), 10), ((45, 540, 14), 10), ((42, 216, 54), 10), ((30, 192, 54), 16),
                                        ((36, 252, 14), 22)])
@pytest.mark.parametrize("bound", [None, 0.7])
def test_wide_tiles(dims, inner, bound):
    base.test_tv_bscan_tiles(dims, inner, bound)


def test_objective_on_wide_tiles():
    base.test_tv_objective_uses_its_own_tiles((45, 216, 30), 10)
