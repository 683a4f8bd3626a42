"""Planes with both sides of 33-64 samples: the reverse sweep from row masks has the bits that the same mapping has from pass
outputs, whichever mapping wrote them, and finds out by itself which of the two a workspace holds."""
import itertools

import numpy as np
import pytest

from gpuutil import run_2d

pytestmark = pytest.mark.gpu

KNOBS = ("plane_per_group64_planes", "plane_per_group64_planes_k2", "plane_per_group64_full_planes_k2",
         "plane_per_group64_full_planes_k3", "plane_per_group64_full_planes_k5", "pair_2d_planes", "pair_2d_many_planes",
         "plane_per_group64_bwd_planes", "plane_per_group64_bwd_ragged_planes", "plane_per_group64_bwd_ragged_planes_k2",
         "fused_keeps_passes")


@pytest.fixture
def overrides():
    import paper_2204_03643_amd as tv
    saved = {k: tv.tv_dispatch_threshold(k) for k in KNOBS}

    def set_to(**values):
        for name, value in values.items():
            tv.tv_dispatch_override(name, value)
    yield set_to
    for name, value in saved.items():
        tv.tv_dispatch_override(name, value)


def _case(H, W, n=5):
    rng = np.random.default_rng(100 * H + W)
    y = np.round(rng.normal(size=(n, H, W)), 1).astype(np.float32)
    return y, (10 ** rng.uniform(-2, 0.5, size=3)).astype(np.float32), rng.normal(size=y.shape).astype(np.float32)


SIDES = [(33, 33), (33, 40), (40, 40), (41, 48), (47, 41), (48, 48), (49, 55), (56, 56), (57, 64), (63, 58), (64, 64)]


@pytest.mark.parametrize("mapping", ["pairs", "planes"])
@pytest.mark.parametrize("H,W", SIDES + [(33, 64), (64, 36)])
def test_masks_and_passes(H, W, mapping, overrides):
    big = 1 << 40
    pairs, group = (0, big) if mapping == "pairs" else (big, big)
    overrides(plane_per_group64_planes=group, plane_per_group64_planes_k2=group, plane_per_group64_full_planes_k2=pairs,
              plane_per_group64_full_planes_k3=pairs, pair_2d_planes=pairs, pair_2d_many_planes=pairs)
    y, lam, g = _case(H, W)
    for K in (1, 2, 3):
        kept = run_2d(y, lam, K, g, keep_passes=True)
        lean = run_2d(y, lam, K, g, keep_passes=False)
        for k in ("x", "gy", "gl"):
            assert np.isfinite(kept[k]).all()
            if k == "x":
                assert np.array_equal(kept[k], lean[k]), (K, k)
            else:                               # (the mapping of the reverse sweep may be another one)
                assert np.abs(kept[k] - lean[k]).max() <= 2e-5 * (1 + np.abs(kept[k]).max()), (K, k)


@pytest.mark.parametrize("H,W", SIDES)
def test_every_writer_with_every_reader(H, W, overrides):
    import torch

    import paper_2204_03643_amd as tv
    big, K = 1 << 40, 2
    y, lam, g = _case(H, W, 3)
    yt, lt, gt = (torch.from_numpy(a).cuda() for a in (y, lam, g))
    L = tv.tv_lambda(lt.data_ptr(), 3, 1)
    wsb = tv.tv2d_workspace_bytes(3, H, W, K)
    ws = torch.full((wsb,), 0xff, dtype=torch.uint8, device="cuda")     # one workspace for all: nothing stale may be believed
    first = {}
    for writer, keep, reader in itertools.product(("pairs", "planes", "passes"), (0, 1), ("pairs", "planes", "passes")):
        group, pairs = {"pairs": (big, 0), "planes": (big, big), "passes": (0, big)}[writer]
        overrides(fused_keeps_passes=keep, plane_per_group64_planes_k2=group, plane_per_group64_full_planes_k2=pairs,
                  pair_2d_planes=pairs, pair_2d_many_planes=pairs)
        x, gy, gl = torch.empty_like(yt), torch.empty_like(yt), torch.empty_like(lt)
        tv.tv2d_prox_fwd(yt, x, 3, H, W, L, K, ws, wsb)
        # another route by the time of the reverse sweep, so that it looks for the other thing
        overrides(fused_keeps_passes=1, plane_per_group64_bwd_planes=0 if reader == "pairs" else big,
                  plane_per_group64_bwd_ragged_planes_k2=big if reader == "planes" else 0)
        tv.tv2d_prox_bwd(gt, gy, gl, 3, H, W, L, K, ws, wsb)
        # masks or pass outputs: the same segments, and the same bits from one reader
        for a, b in zip((x, gy, gl), first.setdefault((writer, reader), (x, gy, gl))):
            assert torch.isfinite(a).all() and torch.equal(a, b), (writer, keep, reader)
        # another reader rounds its means differently
        want = first.setdefault(writer, (x, gy, gl))
        assert torch.equal(x, want[0])
        for a, b in zip((gy, gl), want[1:]):
            assert (a - b).abs().max() <= 2e-5 * (1 + b.abs().max()), (writer, keep, reader)


@pytest.mark.parametrize("lam", [0.0, 0.3])
@pytest.mark.parametrize("H,W", SIDES)
def test_samples_that_are_no_numbers(H, W, lam, overrides):
    """Infinities side by side, zeros of both signs and NaN: the masks say what comparisons of the pass outputs say."""
    import torch

    import paper_2204_03643_amd as tv
    big, K = 1 << 40, 2
    y, _, g = _case(H, W, 4)
    y[0, 5, 3:9], y[1, 7:11, 20], y[2, ::2], y[2, ::2, 1::3] = np.inf, -np.inf, 0.0, -0.0
    y[3, 5, 3], y[3, 9, 7:9], y[3, 20, 20] = np.nan, 3e38, np.inf
    yt, lt, gt = (torch.from_numpy(a).cuda() for a in (y, np.full(4, lam, np.float32), g))
    L = tv.tv_lambda(lt.data_ptr(), 4, 1)
    wsb = tv.tv2d_workspace_bytes(4, H, W, K)
    ws = torch.full((wsb,), 0xff, dtype=torch.uint8, device="cuda")

    def run(writer, keep, reader):
        group, pairs = {"pairs": (big, 0), "planes": (big, big)}[writer]
        overrides(fused_keeps_passes=keep, plane_per_group64_planes_k2=group, plane_per_group64_full_planes_k2=pairs,
                  pair_2d_planes=pairs, pair_2d_many_planes=pairs)
        x, gy, gl = torch.empty_like(yt), torch.empty_like(yt), torch.empty_like(lt)
        tv.tv2d_prox_fwd(yt, x, 4, H, W, L, K, ws, wsb)
        overrides(fused_keeps_passes=1, plane_per_group64_bwd_planes=0 if reader == "pairs" else big,
                  plane_per_group64_bwd_ragged_planes_k2=big if reader == "planes" else 0)
        tv.tv2d_prox_bwd(gt, gy, gl, 4, H, W, L, K, ws, wsb)
        return [t.cpu().numpy() for t in (x, gy, gl)]

    for writer in ("pairs", "planes"):
        for reader in ("planes", "passes"):
            for a, b in zip(run(writer, 1, reader), run(writer, 0, reader)):
                assert np.array_equal(a, b, equal_nan=True), (writer, reader)
        for a, b in zip(run(writer, 0, "passes"), run(writer, 0, "pairs")):
            same = np.isfinite(a)
            assert np.array_equal(same, np.isfinite(b))
            assert np.abs(a[same] - b[same]).max() <= 2e-5 * (1 + np.abs(a[same]).max()), writer


@pytest.mark.parametrize("planes,H,W,K,masks", [(1000, 49, 56, 2, 1), (1300, 49, 56, 2, 0), (1300, 36, 40, 2, 0), (1300, 36, 40, 3, 1), (1300, 41, 48, 3, 0),
                                                (1300, 41, 48, 4, 1), (1300, 47, 47, 3, 1), (5200, 47, 47, 2, 1), (2000, 60, 60, 4, 1), (2600, 60, 60, 4, 0),
                                                (2600, 64, 60, 4, 1), (2100, 58, 64, 6, 0), (2600, 57, 58, 3, 0), (1300, 56, 56, 2, 1)])
def test_one_launch_or_pass_by_pass(planes, H, W, K, masks):
    """Which way forward calls go by default, as the workspace tells it; either way the reverse sweep finds what it needs."""
    import torch

    import paper_2204_03643_amd as tv
    y = torch.randn(planes, H, W, device="cuda", generator=torch.Generator(device="cuda").manual_seed(planes))
    g = torch.randn(planes, H, W, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    lam = torch.tensor([0.3], device="cuda")
    L = tv.tv_lambda(lam.data_ptr(), 1, 1)
    out = []
    for n in (planes, 300):                      # (300: a plane per workgroup)
        wsb = tv.tv2d_workspace_bytes(n, H, W, K)
        ws = torch.full((wsb,), 0xff, dtype=torch.uint8, device="cuda")
        x, gy = torch.empty_like(y[:n]), torch.empty_like(y[:n])
        tv.tv2d_prox_fwd(y, x, n, H, W, L, K, ws, wsb)
        assert int(ws[-16:-12].view(torch.int32)) == (masks if n == planes else 1)
        tv.tv2d_prox_bwd(g, gy, None, n, H, W, L, K, ws, wsb)
        out.append((x[:300], gy[:300]))
    (x, gy), (x1, gy1) = out
    assert (x - x1).abs().max() <= 2e-5 * (1 + y.abs().max())
    # a jump of rounding size more or less moves gradients inside a segment: all but a few agree
    assert ((gy - gy1).abs() > 1e-4 * g.abs().max()).float().mean() < 1e-3


def test_lines_restored_before_the_reverse_sweep(overrides):
    """Masks from a forward call whose line was moved, and moved back by the time of the reverse sweep: it still looks for them."""
    import torch

    import paper_2204_03643_amd as tv
    planes, H, W, K = 600, 40, 64, 1                # by default pass by pass, which leaves pass outputs
    gen = torch.Generator(device="cuda").manual_seed(3)
    y, g = (torch.randn(planes, H, W, device="cuda", generator=gen) for _ in range(2))
    lam = torch.tensor([0.3], device="cuda")
    L = tv.tv_lambda(lam.data_ptr(), 1, 1)
    wsb = tv.tv2d_workspace_bytes(planes, H, W, K)
    default, out = tv.tv_dispatch_threshold("plane_per_group64_planes"), []
    for line, masks in ((default, 0), (1 << 40, 1)):
        ws = torch.full((wsb,), 0xff, dtype=torch.uint8, device="cuda")
        x, gy, gl = torch.empty_like(y), torch.empty_like(y), torch.empty_like(lam)
        overrides(plane_per_group64_planes=line)
        tv.tv2d_prox_fwd(y, x, planes, H, W, L, K, ws, wsb)
        overrides(plane_per_group64_planes=default)
        assert int(ws[-16:-12].view(torch.int32)) == masks
        if masks:
            ws[planes * max(H, W) * 32:-64] = 0xff                  # (no pass outputs to read instead)
        tv.tv2d_prox_bwd(g, gy, gl, planes, H, W, L, K, ws, wsb)
        assert torch.isfinite(gy).all() and torch.isfinite(gl).all()
        out.append((x, gy))
    assert (out[0][0] - out[1][0]).abs().max() <= 2e-5 * (1 + y.abs().max())
    assert ((out[0][1] - out[1][1]).abs() > 1e-4 * g.abs().max()).float().mean() < 1e-3
