"""GPU parity of the kernels that solve a row with two lanes, one from each end (planes of 17-32 samples
a side in one launch), at the sizes where their parts meet: rows that fill the two halves, that lack a
sample or a few, that lie in one half only, and ties across the middle of the row."""
import numpy as np
import pytest

from gpuutil import run_2d
from parity import check_2d

pytestmark = pytest.mark.gpu


@pytest.fixture
def no_plane_per_workgroup():
    import paper_2204_03643_amd as tv
    saved = tv.tv_dispatch_threshold("plane_per_group_planes")
    tv.tv_dispatch_override("plane_per_group_planes", 0)
    yield
    tv.tv_dispatch_override("plane_per_group_planes", saved)


# (halves of 10, 12, 14 and 16 samples: rows of 20, 24, 28 and 32, and their neighbours)
@pytest.mark.parametrize("H,W", [(17, 17), (19, 18), (20, 20), (20, 17), (21, 21), (24, 24), (23, 22), (25, 28), (28, 28),
                                 (27, 26), (29, 32), (30, 30), (31, 31), (32, 32), (32, 31), (32, 16), (17, 32), (32, 15),
                                 (5, 20), (24, 12), (28, 1), (1, 19), (32, 2)])
def test_planes_of_17_to_32_a_side(H, W, no_plane_per_workgroup):
    rng = np.random.default_rng(1000 * H + W)
    y = rng.normal(size=(9, H, W)).astype(np.float32)
    y[3:6] = np.maximum(np.round(y[3:6], 1), 0)               # ties, across the middle too
    y[6:] = np.round(np.cumsum(0.3 * y[6:], axis=2), 1)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.array([0.2, 0.013, 1.7, 0.5], np.float32)
    check_2d(y, lam, 3, g, run_2d(y, lam, 3, g), "pairs %dx%d" % (H, W))
