"""Calls on either side of the dispatch rules that look at a plane's shape or at how rows lie, forced onto small
batches through the thresholds, against the oracle."""
import numpy as np
import pytest

from gpuutil import lam_per_row, run_2d
from parity import check_2d, check_batch

pytestmark = pytest.mark.gpu


@pytest.fixture
def overrides():
    import paper_2204_03643_amd as tv
    saved = tv.tv_dispatch_thresholds()

    def set_to(**values):
        for name, value in values.items():
            tv.tv_dispatch_override(name, value)
    yield set_to
    for name, value in saved.items():
        tv.tv_dispatch_override(name, value)


def _planes(shape):
    rng = np.random.default_rng(shape[0] * 10000 + shape[1] * 100 + shape[2])
    y = rng.normal(size=shape).astype(np.float32)
    y[1::3] = np.maximum(np.round(y[1::3], 1), 0)
    return y, (10 ** rng.uniform(-2, 0.3, size=3)).astype(np.float32), rng.normal(size=shape).astype(np.float32)


@pytest.mark.parametrize("one_launch", [False, True])
@pytest.mark.parametrize("shape", [(70, 1, 17), (33, 4, 32), (40, 32, 3), (21, 16, 17), (9, 32, 16), (12, 15, 32), (10, 20, 28),
                                   (7, 17, 18), (5, 30, 32), (6, 29, 32)])
def test_one_sweep_on_planes_of_at_most_32(shape, one_launch, overrides):
    """One sweep in one launch and pass by pass: thin planes, planes that nearly fill their square (30 x 32) and the
    next that do not (29 x 32)."""
    value = (1 << 40) if one_launch else 0
    overrides(plane_per_group_planes=0, fused32_ragged_planes=value, fused32_full_planes=value)
    y, lam, g = _planes(shape)
    check_2d(y, lam, 1, g, run_2d(y, lam, 1, g), "%s one launch: %s" % (shape, one_launch))


@pytest.mark.parametrize("shape,K", [((3, 40, 40), 1), ((3, 36, 44), 2), ((2, 48, 41), 1), ((2, 56, 56), 2), ((2, 52, 56), 2),
                                     ((2, 55, 50), 4), ((2, 64, 64), 2), ((2, 63, 63), 3), ((2, 60, 64), 3)])
def test_planes_of_33_to_64(shape, K, overrides):
    """Planes that two lanes a row can take: by the rule that gives them to that kernel, and to the others."""
    big = 1 << 40
    y, lam, g = _planes(shape)
    outs = []
    for group, pairs in ((big, 0), (big, big), (0, big)):       # two lanes a row, a plane per workgroup, pass by pass
        overrides(plane_per_group64_planes=group, plane_per_group64_planes_k2=group, plane_per_group64_full_planes_k2=pairs,
                  plane_per_group64_full_planes_k3=pairs, pair_2d_planes=pairs, pair_2d_many_planes=pairs)
        out = run_2d(y, lam, K, g)
        check_2d(y, lam, K, g, out, "%s K=%d group %d pairs %d" % (shape, K, group > 0, pairs == 0))
        outs.append(out["x"])
    # every mapping solves the same problems to rounding
    for x in outs[1:]:
        assert np.abs(x - outs[0]).max() <= 2e-5 * (1 + np.abs(y).max())


@pytest.mark.parametrize("value", [0, 1 << 40])
@pytest.mark.parametrize("n", [33, 40, 41, 57, 64])
def test_rows_that_lie_apart(n, value, overrides):
    """Unit-stride rows with gaps between them, on both sides of the length and of the count from which two lanes
    hold such a row; the gaps stay as they were."""
    import torch

    import paper_2204_03643_amd as tv
    overrides(pair_1d_long_rows=value)
    rng = np.random.default_rng(n)
    y = rng.normal(size=(70, n)).astype(np.float32)
    y[::3] = np.round(y[::3], 1)
    lam = (10 ** rng.uniform(-2, 0.7, size=5)).astype(np.float32)
    spread = np.full((70, n + 3), np.nan, np.float32)
    spread[:, :n] = y
    yt, lt = torch.from_numpy(spread).cuda(), torch.from_numpy(lam).cuda()
    x = torch.full_like(yt, 7.0)
    tv.tv1d_prox_fwd(yt, x, tv.tv_rows(1, 70 * (n + 3), 70, n + 3, n, 1), tv.tv_lambda(lt.data_ptr(), 5, 2))
    out = x.cpu().numpy()
    assert (out[:, n:] == 7.0).all()
    check_batch(y, lam_per_row(lam, 70, 2), None, out[:, :n], None, label="rows of %d apart" % n)


@pytest.mark.parametrize("n,layout,line", [(17, "packed", 160), (20, "packed", 160), (21, "packed", 240), (29, "packed", 400),
                                           (32, "packed", 400), (17, "columns", 120), (31, "columns", 300), (28, "apart", 320),
                                           (29, "apart", 800), (32, "apart", 800)])
def test_line_of_two_lanes_a_row(n, layout, line, overrides):
    """Rows of 17-32 samples at and beyond the count from which two lanes hold a row (pair_1d_rows at 400): the bits are those
    of the mapping that the count asks for, and either mapping's are the oracle's."""
    import torch

    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(n)
    for count in (line, line + 1):
        y = rng.normal(size=(count, n)).astype(np.float32)
        lam = torch.full((1,), 0.7, device="cuda")
        if layout == "columns":
            yt, rows = torch.from_numpy(np.ascontiguousarray(y.T)).cuda(), tv.tv_rows(1, count * n, count, 1, n, count)
        else:
            pitch = n + (3 if layout == "apart" else 0)
            spread = np.zeros((count, pitch), np.float32)
            spread[:, :n] = y
            yt, rows = torch.from_numpy(spread).cuda(), tv.tv_rows(1, count * pitch, count, pitch, n, 1)
        outs = {}
        for value in (0, 400, 1 << 40):
            overrides(pair_1d_rows=value)
            x = torch.zeros_like(yt)
            tv.tv1d_prox_fwd(yt, x, rows, tv.tv_lambda(lam.data_ptr(), 1, 1))
            outs[value] = x.cpu().numpy()
            got = outs[value].T if layout == "columns" else outs[value][:, :n]
            check_batch(y, np.full(count, 0.7, np.float32), None, np.ascontiguousarray(got), None,
                        label="%s rows of %d, pair_1d_rows %d" % (layout, n, value))
        assert not np.array_equal(outs[0], outs[1 << 40])
        assert np.array_equal(outs[400], outs[1 << 40] if count == line else outs[0])
