"""Rows and lambdas of small and of large magnitude: with both multiplied by a power of two the solution is
multiplied by it, also where squares of the values underflow fp32.  Where they are subnormal in part, or
overflow, a row may run into the step cap, but never reports a point as optimal that is not."""
import numpy as np
import pytest

import oracle
from gpuutil import rows_view, run_1d, run_2d

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float32).eps


@pytest.mark.parametrize("power", [-100, -80, -72, -64, -56, -40, -20, 20, 40, 56])
@pytest.mark.parametrize("n,axis", [(32, -1), (64, -1), (100, 0), (256, -1), (512, -1), (700, 0), (900, 0), (1500, -1), (1100, 0),
                                    (5000, -1)])
def test_scaled_rows(n, axis, power):
    rng = np.random.default_rng(n + 7)
    y = np.empty((24, n), np.float32)
    for r in range(24):
        level = np.repeat(rng.uniform(-1, 1, size=n // 9 + 1), 9)[:n]
        y[r] = (rng.normal(size=n), np.round(rng.normal(size=n), 1), level + rng.normal(0, 0.2, size=n),
                np.cumsum(rng.normal(size=n)))[r % 4]
    lam = (10 ** rng.uniform(-1.5, 1.0, size=24)).astype(np.float32)
    s = np.float32(2.0 ** power)
    data = (y if axis == -1 else np.ascontiguousarray(y.T)) * s
    out = run_1d(data, lam * s, 1, axis=axis, want_info=True)
    x = rows_view(out["x"], axis).astype(np.float64) / float(s)
    ref = oracle.prox1d_batch(y.astype(np.float64), lam.astype(np.float64), lam_div=1)
    # the solver's own rounding floor of a difference of two x values
    floor = 16 * EPS * (np.abs(y).max(axis=1) + lam)
    err = np.abs(x - ref).max(axis=1) / floor
    must = np.ones(24, bool)
    if power in (-80, -72, 56):
        must = (out["info"] & (1 << 16)) != 0
        assert must.sum() >= 12
    assert np.all(err[must] <= 1.0), (err.max(), err.argmax(), [hex(i) for i in out["info"][~(err <= 1.0)]])


@pytest.mark.parametrize("power", [-100, -80, -64, -40, 40, 56])
@pytest.mark.parametrize("H,W", [(24, 20), (48, 40), (70, 90)])
def test_scaled_planes(H, W, power):
    """... and where a pass starts from the dual that the correction term encodes (second sweep)."""
    rng = np.random.default_rng(H)
    y = (np.repeat(np.repeat(rng.uniform(-1, 1, size=(4, H // 6 + 1, W // 6 + 1)), 6, 1), 6, 2)[:, :H, :W]
         + rng.normal(0, 0.3, size=(4, H, W))).astype(np.float32)
    lam = np.array([0.05, 0.3, 1.0, 6.0], np.float32)
    s = np.float32(2.0 ** power)
    x = run_2d(y * s, lam * s, 2)["x"].astype(np.float64) / float(s)
    ref, _ = oracle.prox2d_fwd(y.astype(np.float64), lam.astype(np.float64), 2)
    # (four passes, each off by its floor at most, and a prox does not stretch distances: 2-norm)
    floor = 4 * 16 * EPS * (np.abs(y).max(axis=(1, 2)) + 2 * lam) * np.sqrt(H * W)
    err = np.sqrt(((x - ref) ** 2).sum(axis=(1, 2))) / floor
    assert np.all(err <= 1.0), err
