"""3-D TV prox at volumes that take the walk along y with several passes (the small ones of
test_gpu_tv_volume.py step in two kernels): mixes of 1, 2 and 3 steps per pass, one sample past
full tiles in depth and laterally, runs of planes that do not divide n_y, batches; and volumes on
either side of the rule.  Against the FP64 oracle at the tolerance of that file (1e-5)."""
import pytest

import test_gpu_tv_volume as base

pytestmark = pytest.mark.gpu

CASES = [
    ((256, 40, 45, 1), 7), ((256, 40, 45, 1), 10),    # 3 + 2 + 2, 3 + 3 + 2 + 2; the step more: 3 + 3 + 2, 3 + 3 + 3 + 2
    ((175, 54, 35, 1), 5), ((120, 75, 48, 2), 8),     # one sample past three depth tiles, full lateral ones; batches
    ((60, 18, 200, 3), 10), ((135, 40, 7, 5), 4),     # long runs of planes; 4 = 2 + 2
    ((2048, 8, 8, 1), 5), ((1024, 1, 32, 1), 10), ((64, 64, 1, 1), 6), ((512, 20, 20, 1), 9),   # two kernels per step
]


@pytest.mark.parametrize("dims,inner", CASES)
@pytest.mark.parametrize("bound", [None, 0.7])
def test_tv_volume_prox_by_route(dims, inner, bound):
    base.test_tv_volume_prox(dims, inner, bound)
