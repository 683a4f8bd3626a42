"""Small batches of unit-stride rows of 65-256 samples: four samples per thread, against the oracle."""
import numpy as np
import pytest

from gpuutil import run_1d
from parity import check_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 66, 96, 127, 128, 129, 130, 193, 255, 256])
@pytest.mark.parametrize("rows", [1, 37])
def test_four_samples_a_thread(n, rows):
    """Both ends of the two mappings, one row (half a workgroup at up to 128 samples) and an odd count;
    noise, ties and walks, a lambda for each row."""
    import paper_2204_03643_amd as tv
    assert rows <= tv.tv_dispatch_threshold("wave_per_row_rows")
    rng = np.random.default_rng(10 * n + rows)
    y = rng.normal(size=(rows, n)).astype(np.float32)
    y[1::3] = np.round(y[1::3], 1)
    y[2::3] = np.cumsum(y[2::3], axis=1)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = (10 ** rng.uniform(-2, 1, size=rows)).astype(np.float32)
    out = run_1d(y, lam, 1, g, want_info=True)
    check_batch(y, lam, g, out["x"], out["gy"], gl_gpu=out["gl"], lam_count=rows, lam_div=1, label="few rows of %d" % n)
    assert not np.any(out["info"] & (1 << 18))                  # nobody hit the iteration cap
