"""A row's result does not depend on the rows that share its wave or workgroup: the same row alone, in
another order, and between rows that take far longer or hold NaN, bit for bit, for every mapping of
the long-row kernels that puts several rows in a wave; ties included, where the last bit of x
decides what is a segment and with it whole segments of grad_y."""
import numpy as np
import pytest

from gpuutil import rows_view, run_1d, run_2d

pytestmark = pytest.mark.gpu


def _rows(rng, n, count):
    """Rows of noise, 0/1 and one-decimal ties, blocks and random walks in turn, a lambda for each."""
    y = np.empty((count, n), np.float32)
    for r in range(count):
        kind = r % 5
        if kind == 0:
            y[r] = rng.normal(size=n)
        elif kind == 1:
            y[r] = rng.integers(0, 2, size=n)
        elif kind == 2:
            y[r] = np.round(rng.normal(size=n), 1)
        elif kind == 3:
            y[r] = np.round(np.repeat(rng.uniform(-1, 1, size=n // 7 + 1), 7)[:n] + rng.normal(0, 0.1, size=n), 1)
        else:
            y[r] = np.cumsum(rng.normal(size=n))
    lam = rng.choice(np.array([0.05, 0.1, 0.25, 0.5, 1.0, 3.0], np.float32), size=count)
    return y, lam


def _solve(y, lam, g, axis):
    data, up = (y, g) if axis == -1 else (np.ascontiguousarray(y.T), np.ascontiguousarray(g.T))
    out = run_1d(data, lam, 1, up, axis=axis, want_info=True)
    return rows_view(out["x"], axis), rows_view(out["gy"], axis), out["info"]


def _same(got, want, what):
    for q, name in enumerate(("x", "grad_y", "info")):
        differ = np.array([not np.array_equal(a, b) for a, b in zip(got[q], want[q])])
        assert not differ.any(), "%s: %s of %d of %d rows differs" % (what, name, differ.sum(), differ.size)


@pytest.mark.parametrize("n,axis,wide", [(9, -1, 1), (32, -1, 1), (32, -1, 0), (31, 0, 1), (23, 0, 0),
                                         (50, -1, 1), (64, 0, 1), (90, -1, 1), (96, 0, 1), (128, -1, 1), (101, 0, 1),
                                         (190, -1, 1), (192, 0, 1), (256, -1, 1), (250, 0, 1), (383, -1, 1), (384, 0, 1),
                                         (512, -1, 1), (700, 0, 1), (800, -1, 1), (1400, -1, 1), (1100, 0, 1), (2048, 0, 1), (2500, 0, 1), (4000, 0, 1)])
def test_a_row_alone_permuted_and_in_bad_company(n, axis, wide):
    """wide = 0: rows of at most 32 samples on 8 threads instead of 16."""
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(40 * n + axis)
    count = 120 if n <= 400 else 40
    y, lam = _rows(rng, n, count)
    g = rng.normal(size=y.shape).astype(np.float32)
    saved = tv.tv_dispatch_threshold("thread_per_sample_wide_rows")
    try:
        if not wide:
            tv.tv_dispatch_override("thread_per_sample_wide_rows", 0)
        want = _solve(y, lam, g, axis)
        at = rng.permutation(count)
        got = _solve(y[at], lam[at], g[at], axis)
        _same([a[np.argsort(at)] for a in got], want, "permuted")
        # every second row one that is done at once, still runs long after the others, or holds NaN
        mixed = np.zeros((2 * count, n), np.float32)
        mixed[1::2] = y
        mixed[0::4] = np.cumsum(rng.normal(size=mixed[0::4].shape), axis=1)
        mixed[2::8, n // 2] = np.nan
        ml = np.repeat(lam, 2)
        ml[0::4] = 20.0
        got = _solve(mixed, ml, np.repeat(g, 2, axis=0), axis)
        _same([a[1::2] for a in got], want, "mixed")
        few = np.arange(count) if n <= 128 else np.arange(0, count, 4)
        # (a single column would be a unit-stride row: columns get one of zeros beside them)
        pad = [(0, 1 if axis == 0 else 0), (0, 0)]
        alone = [_solve(np.pad(y[r:r + 1], pad), np.repeat(lam[r:r + 1], 1 + pad[0][1]), np.pad(g[r:r + 1], pad), axis)
                 for r in few]
        _same([np.concatenate([a[q][:1] for a in alone]) for q in range(3)], [a[few] for a in want], "alone")
    finally:
        tv.tv_dispatch_override("thread_per_sample_wide_rows", saved)


@pytest.mark.parametrize("H,W", [(70, 100), (40, 66), (200, 130)])
def test_a_plane_alone_and_between_others_pass_by_pass(H, W):
    rng = np.random.default_rng(H)
    y = np.round(np.repeat(np.repeat(rng.uniform(-1, 1, size=(6, H // 5 + 1, W // 5 + 1)), 5, 1), 5, 2)[:, :H, :W]
                 + rng.normal(0, 0.1, size=(6, H, W)), 1).astype(np.float32)
    y[3] = np.cumsum(rng.normal(size=(H, W)), axis=1)
    y[5, H // 2, W // 2] = np.nan
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.array([0.2, 0.05, 0.6, 5.0, 0.1, 0.3], np.float32)
    # (two sweeps: with three, a call with one lambda and one with several run different solvers)
    whole = run_2d(y, lam, 2, g)
    for q in (0, 1, 2, 4):
        one = run_2d(y[q:q + 1], lam[q:q + 1], 2, g[q:q + 1])
        for name in ("x", "gy"):
            assert np.array_equal(one[name][0], whole[name][q]), (q, name)
