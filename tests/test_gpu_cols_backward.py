"""Backward along columns of 33-1024 samples, at the edges of the thread mappings for few and for many columns, against the
oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def _piecewise(rng, P, n, W):
    """Segments from one sample to whole columns, and ties of neighbouring levels."""
    p = 10 ** rng.uniform(-3.5, 0.1, size=(P, 1, W))
    at = rng.random((P, n, W)) < p
    ids = np.cumsum(at, axis=1)
    level = rng.integers(-3, 4, size=(P, n + 1, W)).astype(np.float32)
    return np.take_along_axis(level, ids, axis=1)


@pytest.fixture
def columns(request):
    """The mappings for few columns, and those for many (other ones up to 256 samples) on the same small calls."""
    import paper_2204_03643_amd as tv
    line = tv.tv_dispatch_threshold("bwd_few_columns")
    if request.param == "many":
        tv.tv_dispatch_override("bwd_few_columns", 0)
    yield request.param
    tv.tv_dispatch_override("bwd_few_columns", line)


def _lengths(*ns):
    return [(n, kind) for n in ns for kind in (("few", "many") if n <= 256 else ("few",))]


# 3 x 37 columns: groups of columns that span planes, and a last one partly filled; 41 x 41: 53 groups of 32 or 106 of 16, runs of which
# share an XCD, the last ones in launch order
@pytest.mark.parametrize("P,W", [(3, 37), (41, 41)])
@pytest.mark.parametrize("slots", ["one", "plane", "column"])
@pytest.mark.parametrize("n,columns", _lengths(33, 63, 64, 65, 96, 97, 128, 129, 192, 193, 256, 257, 384, 385, 512, 513, 768, 769, 1024),
                         indirect=["columns"])
def test_columns(n, slots, P, W, columns):
    import torch

    import paper_2204_03643_amd as tv

    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    x = _piecewise(rng, P, n, W)
    g = rng.normal(size=x.shape).astype(np.float32)
    count, div = {"one": (1, 1), "plane": (P, W), "column": (P * W, 1)}[slots]
    xt, gt = torch.from_numpy(x).to(dev), torch.from_numpy(g).to(dev)
    lam = torch.ones(count, device=dev)
    rows, L = tv.rows_along(x.shape, 1), tv.tv_lambda(lam.data_ptr(), count, div)
    room = torch.full((x.size + 64,), float("nan"), device=dev)
    gy, gl = room[32:32 + x.size], torch.full((count,), float("nan"), device=dev)
    wsb = tv.tv1d_bwd_workspace_bytes(rows, L)
    ws = torch.full((max(16, wsb),), 0xff, dtype=torch.uint8, device=dev)
    tv.tv1d_prox_bwd(gt, xt, gy, gl, rows, L, ws, wsb)
    torch.cuda.synchronize()
    assert torch.isnan(room[:32]).all() and torch.isnan(room[32 + x.size:]).all()
    want, wl = oracle.prox1d_bwd_batch(g, x, lam_count=count, axis=1, lam_div=div)
    # sums and means in 64 bits: what shows is the rounding of the mean to a float
    mean_err = 2.0 ** -40 * np.abs(g).max()
    assert (np.abs(gy.cpu().numpy().reshape(x.shape) - want) <= EPS * np.abs(want) + mean_err).all()
    # a slot: a float from every thread with a jump, in each the terms that lie in its chunk and a mean at either end; a float a
    # column where columns do not leave in groups; and the slot's own
    jump = np.diff(x, axis=1) != 0
    terms = (np.abs(np.diff(want, axis=1)) * jump).sum(1).reshape(-1)
    jumps = jump.sum(1).reshape(-1)
    largest = np.abs(want).max(1).reshape(-1)
    slot = (np.arange(P * W) // div) % count
    bound = np.zeros(count)
    np.add.at(bound, slot, EPS * (2 * terms + 2 * np.minimum(jumps, 64) * largest) + 2 * jumps * mean_err)
    assert (np.abs(gl.cpu().numpy() - wl) <= 1.01 * bound + EPS * np.abs(wl)).all()


@pytest.mark.parametrize("n,columns", _lengths(40, 100, 200, 300, 1000), indirect=["columns"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -3e38])
def test_one_bad_sample_stays_in_its_segment(n, bad, columns):
    import torch

    import paper_2204_03643_amd as tv

    rng = np.random.default_rng(n)
    x = _piecewise(rng, 1, n, 21)
    g = rng.normal(size=x.shape).astype(np.float32)
    for k in (0, n // 2, n - 1):
        h = g.copy()
        h[0, k, 3::5] = bad
        want, _ = oracle.prox1d_bwd_batch(np.where(np.isfinite(h) & (np.abs(h) < 1e30), h, 0), x, axis=1)
        same = np.cumsum(np.pad(np.diff(x, axis=1) != 0, ((0, 0), (1, 0), (0, 0))), axis=1)
        hit = np.zeros(x.shape, bool)
        hit[0, :, 3::5] = (same == same[:, k:k + 1])[0, :, 3::5]
        xt, ht = torch.from_numpy(x).cuda(), torch.from_numpy(h).cuda()
        lam = torch.ones(1, device="cuda")
        rows, L = tv.rows_along(x.shape, 1), tv.tv_lambda(lam.data_ptr(), 1, 1)
        gy = torch.empty_like(ht)
        tv.tv1d_prox_bwd(ht, xt, gy, None, rows, L, None, 0)
        got = gy.cpu().numpy()
        assert (np.abs(got - want) <= EPS * np.abs(want) + 2.0 ** -40 * np.abs(g).max())[~hit].all()
        if bad != -3e38:
            assert not np.isfinite(got[hit]).any()


def _lambda_grads(x, g, count, div):
    import torch

    import paper_2204_03643_amd as tv
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    lam = torch.ones(count, device="cuda")
    rows, L = tv.rows_along(x.shape, 1), tv.tv_lambda(lam.data_ptr(), count, div)
    gy, gl = torch.empty_like(gt), torch.full((count,), float("nan"), device="cuda")
    wsb = tv.tv1d_bwd_workspace_bytes(rows, L)
    ws = torch.full((max(16, wsb),), 0xff, dtype=torch.uint8, device="cuda")
    tv.tv1d_prox_bwd(gt, xt, gy, gl, rows, L, ws, wsb)
    return gl.cpu().numpy()


@pytest.mark.parametrize("n,columns", _lengths(40, 100, 200, 300, 1000), indirect=["columns"])
@pytest.mark.parametrize("bad", [float("inf"), -float("inf"), 3e38])
def test_an_infinite_lambda_gradient(n, bad, columns):
    """A slot whose terms add up to an infinity has it as its gradient, whether one column or many share the slot."""
    W = 64
    x = np.zeros((1, n, W), np.float32)
    x[0, n // 2:] = 1                               # one rise: the gradient is the sum of the lower halves' means less the upper ones'
    g = np.ones(x.shape, np.float32)
    if np.isinf(bad):
        g[0, n // 4, 3] = bad
    else:
        g[0, :n // 2] = bad                         # (every column's term is a float, the sum of two is not)
    want = np.float32(np.sign(bad) * np.inf)
    assert _lambda_grads(x, g, 1, 1)[0] == want
    assert np.array_equal(_lambda_grads(x, g, 4, 16), [want] + ([0] * 3 if np.isinf(bad) else [want] * 3))


@pytest.mark.parametrize("n,columns", _lengths(40, 100, 200, 300, 1000), indirect=["columns"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_bad_segment_on_a_staircase_shows(n, bad, columns):
    """Between two rises a segment's mean enters once with either sign: an infinity or NaN there leaves NaN, wherever the segment
    lies in its thread's chunk."""
    W = n - 8
    x = np.repeat((np.arange(n) // 2).astype(np.float32)[:, None], W, 1)[None]
    g = np.ones(x.shape, np.float32)
    at = np.arange(W)
    g[0, at + 4, at] = bad
    assert np.isnan(_lambda_grads(x, g, W, 1)).all()
    assert np.isnan(_lambda_grads(x, g, 1, 1)).all()


@pytest.mark.parametrize("n", [33, 40, 44, 48, 50, 57, 60, 63, 64])
def test_many_short_columns_with_and_without_a_lambda_gradient(n):
    """More than 16 384 columns: the kernel that forms no dL/dlam has the bits of the one that does, and both are right where
    the column's end cuts a thread's chunk."""
    import torch

    import paper_2204_03643_amd as tv
    P, W = 410, 41
    rng = np.random.default_rng(n)
    x = _piecewise(rng, P, n, W)
    g = rng.normal(size=x.shape).astype(np.float32)
    want, wl = oracle.prox1d_bwd_batch(g, x, lam_count=P, axis=1, lam_div=W)
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    lam = torch.ones(P, device="cuda")
    rows, L = tv.rows_along(x.shape, 1), tv.tv_lambda(lam.data_ptr(), P, W)
    wsb = tv.tv1d_bwd_workspace_bytes(rows, L)
    ws = torch.full((wsb,), 0xff, dtype=torch.uint8, device="cuda")
    out = []
    for gl in (torch.empty(P, device="cuda"), None):
        room = torch.full((x.size + 64,), float("nan"), device="cuda")
        gy = room[32:32 + x.size]
        tv.tv1d_prox_bwd(gt, xt, gy, gl, rows, L, ws, wsb)
        assert torch.isnan(room[:32]).all() and torch.isnan(room[32 + x.size:]).all()
        out.append((gy.cpu().numpy().reshape(x.shape), gl))
    assert np.array_equal(out[0][0], out[1][0])
    # a mean is a float of a sum in 64 bits; a slot adds up in 64 bits a float from each of W x 4 threads, in each the terms that lie
    # in its chunk and a mean at either end
    assert np.abs(out[0][0] - want).max() <= 2 * EPS * np.abs(g).max()
    terms = np.abs(np.diff(want, axis=1)) * (np.diff(x, axis=1) != 0)
    bound = EPS * (terms.sum((1, 2)) + W * 4 * 2 * np.abs(want).max((1, 2)) + np.abs(wl))
    assert (np.abs(out[0][1].cpu().numpy() - wl) <= 1.01 * bound).all()
