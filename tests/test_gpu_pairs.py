"""GPU parity of the kernels that solve a row with two lanes, one from each end (1D rows of 17-64 samples
in large batches; planes of 17-64 samples a side in one launch), at the sizes where their parts meet:
rows that fill the two halves, that lack a sample or a few, that lie in one half only, ties across the
middle of the row, and every way the rows can lie in memory."""
import numpy as np
import pytest

from gpuutil import lam_per_row, run_2d
from parity import check_2d, check_batch

pytestmark = pytest.mark.gpu


@pytest.fixture
def pairs():
    import paper_2204_03643_amd as tv
    saved = {k: tv.tv_dispatch_threshold(k) for k in ("plane_per_group_planes", "thread_per_sample_1d_rows", "pair_1d_long_rows",
                                                      "plane_per_group64_planes", "plane_per_group64_full_planes_k2",
                                                      "plane_per_group64_full_planes_k3", "pair_2d_planes", "pair_2d_many_planes")}
    for k in saved:
        tv.tv_dispatch_override(k, 0)
    yield
    for k, v in saved.items():
        tv.tv_dispatch_override(k, v)


# (halves of 10, 12, 14 and 16 samples: rows of 20, 24, 28 and 32, and their neighbours)
@pytest.mark.parametrize("H,W", [(17, 17), (19, 18), (20, 20), (20, 17), (21, 21), (24, 24), (23, 22), (25, 28), (28, 28),
                                 (27, 26), (29, 32), (30, 30), (31, 31), (32, 32), (32, 31), (32, 16), (17, 32), (32, 15),
                                 (5, 20), (24, 12), (28, 1), (1, 19), (32, 2),
                                 # halves of 20, 24, 28 and 32, two waves a plane
                                 (33, 33), (40, 40), (33, 39), (40, 32), (41, 41), (48, 48), (47, 40), (39, 45), (49, 52),
                                 (56, 56), (55, 45), (57, 57), (64, 64), (63, 62), (64, 52), (52, 60)])
def test_planes_of_17_to_64_a_side(H, W, pairs):
    rng = np.random.default_rng(1000 * H + W)
    y = rng.normal(size=(9, H, W)).astype(np.float32)
    y[3:6] = np.maximum(np.round(y[3:6], 1), 0)               # ties, across the middle too
    y[6:] = np.round(np.cumsum(0.3 * y[6:], axis=2), 1)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.array([0.2, 0.013, 1.7, 0.5], np.float32)
    check_2d(y, lam, 3, g, run_2d(y, lam, 3, g), "pairs %dx%d" % (H, W))


# how the rows of n lie, as (outer stride, inner stride, element stride) of 7 x 16 rows, in samples:
# packed, packed at a 4-byte offset, rows with gaps, columns, columns with gaps
LAYOUTS = {"packed": lambda n: (16 * n, n, 1, 0), "shifted": lambda n: (16 * n, n, 1, 1), "gaps": lambda n: (20 * (n + 3), n + 3, 1, 0),
           "columns": lambda n: (16 * n, 1, 16, 0), "gap columns": lambda n: (37 * n, 2, 36, 3)}


@pytest.mark.parametrize("n", [17, 18, 19, 20, 21, 23, 24, 25, 27, 28, 29, 30, 31, 32, 33, 36, 39, 40, 41, 47, 48, 49, 53, 56,
                               57, 60, 63, 64])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("count,div", [(1, 1), (112, 1), (7, 16), (2, 8)])
def test_rows_of_17_to_64_in_every_layout(n, layout, count, div, pairs):
    """112 rows (the last wave half empty, except where the rows of a lambda are grouped): output, info
    words, segment codes (up to 32 samples) and both gradients; nothing is written outside the rows."""
    import torch
    import paper_2204_03643_amd as tv
    so, si, se, at = LAYOUTS[layout](n)
    outer = 8 if (count, div) == (2, 8) else 7                # 128 rows: two slots of two whole waves each
    rows_n = outer * 16
    rng = np.random.default_rng(100 * n + count)
    yr = rng.normal(size=(rows_n, n)).astype(np.float32)
    yr[::3] = np.round(yr[::3], 1)
    gr = rng.normal(size=yr.shape).astype(np.float32)
    lam = (10 ** rng.uniform(-2, 0.7, size=count)).astype(np.float32)
    where = at + (np.arange(rows_n) // 16 * so + np.arange(rows_n) % 16 * si)[:, None] + np.arange(n) * se
    size = int(where.max()) + 8
    dev = torch.device("cuda:0")

    def spread(a):
        b = np.full(size, np.nan, np.float32)
        b[where] = a
        return torch.from_numpy(b).to(dev)

    y, g = spread(yr), spread(gr)
    x, gy = torch.full_like(y, np.nan), torch.full_like(y, np.nan)
    lt = torch.from_numpy(lam).to(dev)
    gl = torch.empty_like(lt)
    rows, L = tv.tv_rows(outer, so, 16, si, n, se), tv.tv_lambda(lt.data_ptr(), count, div)
    info = torch.zeros(rows_n, dtype=torch.int32, device=dev)
    seg = torch.full((rows_n,), -1, dtype=torch.int64, device=dev)
    wsb = tv.tv1d_bwd_workspace_bytes(rows, L)
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    tv.tv1d_prox_fwd_ex(y[at:], x[at:], rows, L, info=info, seg=seg if n <= 32 else None)
    if n <= 32:
        tv.tv1d_prox_bwd_seg(g[at:], seg, gy[at:], gl, rows, L, ws, wsb)
    else:
        tv.tv1d_prox_bwd(g[at:], x[at:], gy[at:], gl, rows, L, ws, wsb)
    torch.cuda.synchronize()
    out = x.cpu().numpy()
    xr, gyr = out[where], gy.cpu().numpy()[where]
    rest = np.ones(size, bool)
    rest[where] = False
    assert np.isnan(out[rest]).all() and np.isnan(gy.cpu().numpy()[rest]).all()
    if n <= 32:
        code = np.zeros(rows_n, np.uint64)
        for k in range(n - 1):
            code |= (xr[:, k + 1] != xr[:, k]).astype(np.uint64) << np.uint64(k)
            code |= (xr[:, k + 1] > xr[:, k]).astype(np.uint64) << np.uint64(32 + k)
        assert np.array_equal(seg.cpu().numpy().view(np.uint64), code)
    assert not (info.cpu().numpy() >> 18).any()               # no row stopped short
    check_batch(yr, lam_per_row(lam, rows_n, div), gr, xr, gyr, gl_gpu=gl.cpu().numpy(), lam_count=count, lam_div=div,
                label="pairs n=%d %s" % (n, layout))


@pytest.mark.parametrize("div,count", [(32, 2), (8, 4), (1, 32), (16, 2)])
def test_plane_columns_with_several_lambdas_a_plane(div, count, pairs):
    """Columns of 32 x 32 planes whose lambda changes inside a plane: a wave that held the columns of one
    lambda would not hold a plane."""
    import torch
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(div)
    y = rng.normal(size=(8, 32, 32)).astype(np.float32)
    lam = (10 ** rng.uniform(-2, 0.5, size=count)).astype(np.float32)
    yt, lt = torch.from_numpy(y).cuda(), torch.from_numpy(lam).cuda()
    x = torch.full_like(yt, float("nan"))
    tv.tv1d_prox_fwd(yt, x, tv.tv_rows(8, 1024, 32, 1, 32, 32), tv.tv_lambda(lt.data_ptr(), count, div))
    torch.cuda.synchronize()
    cols = lambda a: a.transpose(0, 2, 1).reshape(-1, 32)
    check_batch(cols(y), lam_per_row(lam, 256, div), None, cols(x.cpu().numpy()), None, label="plane columns")


@pytest.mark.parametrize("n,axis", [(33, -1), (40, 0), (48, -1), (55, 0), (64, -1), (64, 0)])
def test_rows_of_33_to_64_alone_in_company_and_scaled(n, axis, pairs):
    """What the other kernels for these lengths promise: a row has the same bits alone, in another order and
    between rows that take longer or hold NaN; lambda = 0 is the identity; and with data and lambda both
    multiplied by a power of two so is the solution, where their squares underflow too."""
    import oracle
    from gpuutil import rows_view, run_1d
    rng = np.random.default_rng(n)
    count = 90
    y = rng.normal(size=(count, n)).astype(np.float32)
    y[::3] = np.round(y[::3], 1)
    y[1::3] = np.cumsum(0.3 * y[1::3], axis=1)
    lam = (10 ** rng.uniform(-1.5, 0.7, size=count)).astype(np.float32)
    turn = lambda a: a if axis == -1 else np.ascontiguousarray(a.T)
    solve = lambda a, l: (lambda o: (rows_view(o["x"], axis), o["info"]))(run_1d(turn(a), l, 1, axis=axis, want_info=True))
    want, info = solve(y, lam)
    at = rng.permutation(count)
    got, gi = solve(y[at], lam[at])
    assert np.array_equal(got, want[at]) and np.array_equal(gi, info[at])
    mixed, ml = np.repeat(y, 2, axis=0), np.repeat(lam, 2)
    mixed[0::4] = np.cumsum(rng.normal(size=mixed[0::4].shape), axis=1)
    mixed[2::8, n // 2] = np.nan
    ml[0::4] = 20.0
    got, gi = solve(mixed, ml)
    assert np.array_equal(got[1::2], want) and np.array_equal(gi[1::2], info)
    for r in range(0, count, 9):
        got, _ = solve(np.stack([y[r], 0 * y[r]]), np.repeat(lam[r], 2))
        assert np.array_equal(got[0], want[r])
    assert np.array_equal(solve(y, np.zeros(1, np.float32))[0], y)
    ref = oracle.prox1d_batch(y.astype(np.float64), lam.astype(np.float64), lam_div=1)
    floor = 16 * np.finfo(np.float32).eps * (np.abs(y).max(axis=1) + lam)         # as the solver's own
    for power in (-100, -64, -40, 0, 20, 40):
        s = np.float32(2.0 ** power)
        x = solve(y * s, lam * s)[0].astype(np.float64) / float(s)
        assert np.all(np.abs(x - ref).max(axis=1) <= floor), power


@pytest.mark.parametrize("n,axis", [(17, -1), (20, 0), (23, -1), (28, 0), (31, -1), (32, -1), (32, 0)])
def test_rows_of_17_to_32_alone_and_in_company(n, axis, pairs):
    """Rows of 17-32 samples on two lanes: a row has the same bits, info word and segment code alone, in another
    order and between rows that take longer, hold a NaN or an infinity; lambda = 0 is the identity."""
    from gpuutil import rows_view, run_1d
    rng = np.random.default_rng(n + 100 * (axis + 1))
    count = 90
    y = rng.normal(size=(count, n)).astype(np.float32)
    y[::3] = np.round(y[::3], 1)
    y[1::3] = np.cumsum(0.3 * y[1::3], axis=1)
    lam = (10 ** rng.uniform(-1.5, 0.7, size=count)).astype(np.float32)
    turn = lambda a: a if axis == -1 else np.ascontiguousarray(a.T)

    def solve(a, l):
        info = run_1d(turn(a), l, 1, axis=axis, want_info=True)
        seg = run_1d(turn(a), l, 1, axis=axis, use_seg=True)
        assert np.array_equal(info["x"], seg["x"], equal_nan=True)
        return rows_view(info["x"], axis), info["info"], seg["seg"]

    want = solve(y, lam)
    at = rng.permutation(count)
    for got, ref in zip(solve(y[at], lam[at]), want):
        assert np.array_equal(got, ref[at])
    mixed, ml = np.repeat(y, 2, axis=0), np.repeat(lam, 2)
    mixed[0::4] = np.cumsum(rng.normal(size=mixed[0::4].shape), axis=1)
    mixed[2::8, n // 2] = np.nan
    mixed[6::8, n // 3] = np.inf
    ml[0::4] = 20.0
    got = solve(mixed, ml)
    for a, ref in zip(got, want):
        assert np.array_equal(a[1::2], ref)
    assert np.isnan(got[0][2::8, n // 2]).all() and not np.isfinite(got[0][6::8, n // 3]).any()
    for r in range(0, count, 9):
        alone = solve(np.stack([y[r], 0 * y[r]]), np.repeat(lam[r], 2))
        for a, ref in zip(alone, want):
            assert np.array_equal(a[0], ref[r])
    assert np.array_equal(solve(y, np.zeros(1, np.float32))[0], y)


@pytest.mark.parametrize("H,W", [(17, 20), (24, 24), (29, 32), (32, 32), (40, 40), (63, 63)])
def test_planes_alone_and_in_company(H, W, pairs):
    """Planes on two lanes a row: a plane has the same bits, gradients too, alone, in another order and beside a
    plane with a NaN."""
    rng = np.random.default_rng(H * 100 + W)
    y = np.maximum(rng.normal(size=(9, H, W)), -0.3).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = (10 ** rng.uniform(-1.5, 0.5, size=9)).astype(np.float32)
    want = run_2d(y, lam, 3, g)
    at = rng.permutation(9)
    got = run_2d(y[at], lam[at], 3, g[at])
    for k in ("x", "gy", "gl"):
        assert np.array_equal(got[k], want[k][at]), k
    alone = run_2d(y[4:5], lam[4:5], 3, g[4:5])
    spoilt = y.copy()
    spoilt[3, H // 2, W // 2] = np.nan
    beside = run_2d(spoilt, lam, 3, g)
    rest = np.arange(9) != 3
    for k in ("x", "gy", "gl"):
        assert np.array_equal(alone[k][0], want[k][4]), k
        assert np.array_equal(beside[k][rest], want[k][rest]), k
    assert np.isnan(beside["x"][3, H // 2, W // 2])


@pytest.mark.parametrize("H,W", [(40, 40), (33, 36), (33, 40), (39, 40), (41, 44), (39, 48), (48, 40), (48, 48), (49, 52),
                                 (45, 56), (56, 56), (57, 60), (52, 64), (64, 52), (63, 64), (64, 64)])
@pytest.mark.parametrize("K", [1, 3])
def test_reverse_sweep_of_planes_of_33_to_64(H, W, K):
    """The one-launch reverse sweep with two lanes a row, both ends of every half length and the most samples
    past a row's end, against the oracle."""
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(H * 100 + W + K)
    y = np.maximum(rng.normal(size=(5, H, W)), -0.3).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = np.array([0.02, 0.3, 1.5], np.float32)
    most = tv.tv_dispatch_threshold("plane_per_group64_bwd_planes")
    tv.tv_dispatch_override("plane_per_group64_bwd_planes", 0)
    try:
        out = run_2d(y, lam, K, g)
    finally:
        tv.tv_dispatch_override("plane_per_group64_bwd_planes", most)
    check_2d(y, lam, K, g, out, "reverse pairs %dx%d" % (H, W))
