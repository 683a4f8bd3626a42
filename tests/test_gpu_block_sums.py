"""GPU parity: the long-row solver's block sums, on rows whose constant blocks span threads, 16-lane
rows, half waves, waves and the whole workgroup, at the row lengths where the mapping changes."""
import numpy as np
import pytest

import oracle
from gpuutil import rows_view, run_1d, run_2d
from parity import check_2d

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float32).eps


def _rows(rng, n):
    """Levels with blocks of 1, a few, a third of n and nearly n samples; small noise, and an offset
    that dwarfs it in half of the rows."""
    y = np.empty((8, n), np.float32)
    for r in range(8):
        size = (1, 5, max(1, n // 3), max(1, n - 2))[r % 4]
        level = np.repeat(rng.uniform(-1.0, 1.0, size=n // size + 1), size)[:n]
        y[r] = level + rng.normal(0, 0.02, size=n) + (100.0 if r >= 4 else 0.0)
    return y


@pytest.mark.parametrize("n", [33, 63, 65, 96, 97, 129, 191, 257, 385, 511, 513, 767, 769, 1023, 1025, 1537, 2049, 3073,
                               4095, 4097, 6145, 8193, 12289, 16383, 16384])
@pytest.mark.parametrize("lam", [0.003, 0.6, 30.0])
def test_blocks_across_threads_and_waves(n, lam):
    rng = np.random.default_rng(9000 + n)
    y = _rows(rng, n)
    lam = np.array([lam], np.float32)
    for axis, data in ((-1, y), (0, np.ascontiguousarray(y.T))):          # packed rows; columns (strided samples)
        out = run_1d(data, lam, 1, axis=axis, want_info=True)
        assert not np.any(out["info"] & ((1 << 18) | (1 << 19)))          # no cap, every row in blocks
        x = rows_view(out["x"], axis)
        ref = oracle.prox1d_batch(y.astype(np.float64), lam.astype(np.float64))
        # the solver's own rounding floor of a difference of two x values, 16 eps (max|y| + lam); a dual
        # that rounding puts on the other side of its bound moves two block means by no more than that
        floor = 16 * EPS * (np.abs(y).max(axis=1) + lam[0])
        assert np.all(np.abs(x - ref).max(axis=1) <= floor), (n, lam, axis, (np.abs(x - ref).max(axis=1) / floor).max())


@pytest.mark.parametrize("H,W", [(65, 100), (33, 130), (200, 257), (513, 70), (769, 40)])
@pytest.mark.parametrize("count", [1, 3])
def test_2d_passes_with_one_and_with_several_lambdas(H, W, count):
    """Three sweeps with one lambda take the passes of their own that keep their rounding."""
    rng = np.random.default_rng(H * W)
    y = (np.repeat(np.repeat(rng.uniform(-1, 1, size=(3, H // 8 + 1, W // 8 + 1)), 8, 1), 8, 2)[:, :H, :W]
         + rng.normal(0, 0.2, size=(3, H, W))).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.array([0.15, 0.02, 0.6], np.float32)[:count]
    check_2d(y, lam, 3, g, run_2d(y, lam, 3, g), "%dx%d, %d lambdas" % (H, W, count))


@pytest.mark.parametrize("H,W", [(65, 100), (200, 257), (513, 70)])
def test_one_lambda_and_the_same_lambda_repeated(H, W):
    """The two solvers agree to rounding; with the threshold at 0 there is one, and the bits agree."""
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(H + W)
    y = (np.repeat(np.repeat(rng.uniform(-1, 1, size=(3, H // 8 + 1, W // 8 + 1)), 8, 1), 8, 2)[:, :H, :W]
         + rng.normal(0, 0.2, size=(3, H, W))).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.full(3, 0.2, np.float32)
    many = run_2d(y, lam, 3, g)
    tri = run_2d(y, lam[:1], 3, g)
    saved = tv.tv_dispatch_threshold("one_lambda_tri_side")
    try:
        tv.tv_dispatch_override("one_lambda_tri_side", 0)
        one = run_2d(y, lam[:1], 3, g)
    finally:
        tv.tv_dispatch_override("one_lambda_tri_side", saved)
    check_2d(y, lam[:1], 3, g, tri, "%dx%d, tridiagonal" % (H, W))
    check_2d(y, lam[:1], 3, g, one, "%dx%d, block means" % (H, W))
    assert np.array_equal(one["x"], many["x"]) and np.array_equal(one["gy"], many["gy"])
    # six passes, each off by its floor at most on both sides; a prox does not stretch distances (2-norm)
    floor = 2 * 6 * 16 * EPS * (np.abs(y).max() + 2 * lam[0]) * np.sqrt(y.size)
    assert np.linalg.norm(tri["x"].astype(np.float64) - one["x"]) <= floor


@pytest.mark.parametrize("n,axis,limit", [(12, -1, 128), (16, -1, 128), (17, -1, 256), (32, -1, 256),
                                          (12, 0, 64), (16, 0, 64), (17, 0, 256), (31, 0, 256), (32, 0, 128)])
def test_short_rows_change_mapping_at_their_row_count(n, axis, limit):
    """With the threshold at 256 rows, shorter rows and columns change over at a half or a quarter of
    it: on either side the result has the bits of the mapping that belongs there.  (That the two
    mappings round differently, without which a wrong threshold would not show, is not asked for.)"""
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(n)
    lam = np.array([0.4], np.float32)
    saved = tv.tv_dispatch_threshold("thread_per_sample_1d_rows")
    try:
        for rows in (limit, limit + 1):
            y = rng.normal(size=(rows, n)).astype(np.float32)
            data = y if axis == -1 else np.ascontiguousarray(y.T)
            x = {}
            for value in (256, 1 << 40, 0):
                tv.tv_dispatch_override("thread_per_sample_1d_rows", value)
                x[value] = rows_view(run_1d(data, lam, 1, axis=axis)["x"], axis)
            assert np.array_equal(x[256], x[1 << 40 if rows == limit else 0])
            ref = oracle.prox1d_batch(y.astype(np.float64), lam.astype(np.float64))
            floor = 16 * EPS * (np.abs(y).max(axis=1) + lam[0])            # as above
            assert np.all(np.abs(x[256] - ref).max(axis=1) <= floor)
    finally:
        tv.tv_dispatch_override("thread_per_sample_1d_rows", saved)


@pytest.mark.parametrize("H,W", [(64, 64), (33, 64), (48, 40)])
def test_2d_planes_of_64_pass_by_pass_with_one_lambda(H, W):
    import paper_2204_03643_amd as tv
    names = ("plane_per_group64_planes_k2", "plane_per_group64_full_planes_k3")
    saved = {k: tv.tv_dispatch_threshold(k) for k in names}
    rng = np.random.default_rng(H + W)
    y = np.maximum(rng.normal(size=(5, H, W)), 0).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.array([0.2], np.float32)
    try:
        for k in names:
            tv.tv_dispatch_override(k, 0)
        check_2d(y, lam, 3, g, run_2d(y, lam, 3, g), "%dx%d" % (H, W))
    finally:
        for k, v in saved.items():
            tv.tv_dispatch_override(k, v)
