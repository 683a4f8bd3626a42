"""The coarse level of long rows forms its averages itself: ragged last groups at every thread mapping, rows that take
part and rows that do not side by side, against the oracle."""
import numpy as np
import pytest

from gpuutil import run_1d
from parity import check_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_ws", [False, True])
@pytest.mark.parametrize("n", [770, 771, 1026, 1027, 1538, 2051, 3074, 4094, 6147, 8194, 12290, 16383])
def test_ragged_groups(n, use_ws):
    rows = 9                                     # (up to eight rows share a workgroup)
    rng = np.random.default_rng(n)
    y = rng.normal(size=(rows, n)).astype(np.float32)
    y[::2] = np.cumsum(0.1 * y[::2], axis=1)
    g = rng.normal(size=y.shape).astype(np.float32)
    # one row in three has a lambda far below its variation
    lam = np.where(np.arange(rows) % 3 == 2, 1e-3, 10 ** rng.uniform(-0.5, 1, size=rows)).astype(np.float32)
    out = run_1d(y, lam, 1, g, want_info=True, use_ws=use_ws)
    check_batch(y, lam, g, out["x"], out["gy"], gl_gpu=out["gl"], lam_count=rows, lam_div=1, label="n=%d" % n)
    assert not np.any(out["info"] & (1 << 18))                  # nobody hit the iteration cap
