"""Interpolated-ISAM fill (Sec. 3.1) where the scan over mask words can go wrong: row lengths
around a word and around the 64 words of a wave, long gaps, a single observed pixel at either
end of the row or of a word, nothing observed.  Against the FP64 oracle (1e-5, the tolerance
of the other direct images)."""
import numpy as np
import pytest

import oracle as O
from gpu_util import both_geoms, flush, rel, to_dev, to_host

pytestmark = pytest.mark.gpu


def _rows(rng, nk):
    """One A-scan per pattern."""
    m = np.zeros((9, nk), np.uint8)
    m[0, 0] = m[1, nk - 1] = m[2, min(31, nk - 1)] = m[3, min(32, nk - 1)] = 1   # single pixels
    m[4, [0, nk - 1]] = 1                                                        # one gap over the row
    m[5, nk // 3: nk // 3 + 2] = 1
    m[6] = rng.random(nk) < 0.5
    m[7] = rng.random(nk) < 0.01
    return m                                                                     # m[8]: nothing observed


@pytest.mark.parametrize("nk", [2, 31, 32, 33, 100, 2047, 2048, 2049, 5000])
def test_interp_fill(nk):
    import paper_2108_01438_amd as P
    flush(f"[interp fill] n_k={nk}")
    rng = np.random.default_rng(nk)
    og, pg = both_geoms(n_depth=32, n_x=9, n_k=nk)
    mask = _rows(rng, nk)[None]
    y = rng.standard_normal(O.meas_shape(og)).astype(np.float32)
    x = to_host(P.Plan(pg, mask).direct(to_dev(y), "interp_isam"))
    assert rel(x, O.interp_isam(y.astype(np.float64), og, mask)) <= 1e-5
