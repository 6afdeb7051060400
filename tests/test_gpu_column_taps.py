"""Windows of 4 and 8 taps in every variant of the column kernels: two base cells per thread
(few pairs), three and five (many), at compiled lengths, run-time ones, and a compiled length whose
columns span more cells than its variant has threads for.  Against the FP64 oracle at the
tolerance of the other operator tests (1e-5)."""
import pytest

import test_gpu_columns as base

pytestmark = pytest.mark.gpu
DZ0 = base.DZ0

CASES = [
    dict(n_depth=512, n_x=9, n_k=520), dict(n_depth=1024, n_x=6, n_k=900), dict(n_depth=2048, n_x=4, n_k=2048),
    dict(n_depth=512, n_x=540, n_k=500), dict(n_depth=1024, n_x=525, n_k=1024),
    dict(n_depth=945, n_x=3, n_k=1003), dict(n_depth=700, n_x=750, n_k=650), dict(n_depth=128, n_x=2100, n_k=120),
    dict(n_depth=2048, n_x=3, n_k=1700, dz=1.7 * DZ0 * 1699 / 2048),
    dict(n_depth=160, n_x=10, n_k=150, z_focus=12.0, disp_b=1e-6),
    dict(n_depth=64, n_x=24, n_k=64, k_min=0.3, k_max=0.9, dx=0.9),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join(f"{k}{v:.4g}" for k, v in kw.items()))
@pytest.mark.parametrize("kb_width", [4, 8])
@pytest.mark.parametrize("masked", [False, True])
def test_taps(kw, kb_width, masked):
    base.test_columns(dict(kw, kb_width=kb_width), masked)
