"""Evanescent samples with a focus off the middle, in units other than rad/um: the empty base
cell beside the cut-off must add nothing, however far below it the sample looked at lies.
Against the FP64 oracle at the tolerance of the other operator tests (1e-5)."""
import pytest

import test_gpu_columns as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("unit", [1.0, 1e3, 1e6], ids=["um", "mm", "m"])
@pytest.mark.parametrize("n_x", [24, 525])
@pytest.mark.parametrize("masked", [False, True])
def test_units(unit, n_x, masked):
    kw = dict(n_depth=80, n_x=n_x, n_k=64, k_min=0.3 * unit, k_max=0.9 * unit, dx=0.9 / unit, z_focus=100.0 / unit,
              beam_waist=0.2 / unit)
    base.test_columns(kw, masked)
