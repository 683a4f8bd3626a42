"""The sum of dL/dlam terms over a slot's rows, at the counts where the threads a slot gets change, against 64 bits; and a
lambda for every row or plane, where the terms are the gradient."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("div", [1, 3, 64])
@pytest.mark.parametrize("per_slot", [1, 2, 3, 8, 9, 32, 33, 128, 129, 2048, 2049, 5000])
def test_rows_per_slot(per_slot, div):
    import torch

    import paper_2204_03643_amd as tv

    n, count = 40, 3                               # (rows of more than 32 samples leave a term each)
    rows = count * per_slot - (1 if per_slot > 2 else 0)           # (the last slot one short)
    rng = np.random.default_rng(per_slot + div)
    x = np.round(rng.normal(size=(rows, n)), 0).astype(np.float32)
    g = rng.normal(size=x.shape).astype(np.float32)
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    lam = torch.ones(count, device="cuda")
    r, L = tv.rows_along(x.shape, -1), tv.tv_lambda(lam.data_ptr(), count, div)
    gy, gl = torch.empty_like(gt), torch.full((count,), float("nan"), device="cuda")
    wsb = tv.tv1d_bwd_workspace_bytes(r, L)
    ws = torch.full((max(16, wsb),), 0xff, dtype=torch.uint8, device="cuda")
    tv.tv1d_prox_bwd(gt, xt, gy, gl, r, L, ws, wsb)
    gy64, want = oracle.prox1d_bwd_batch(g, x, lam_count=count, lam_div=div)
    # a term: at most 39 jumps, each the difference of two means of |g| <= 6, within some 20 ulp of one
    slot = (np.arange(rows) // div) % count
    bound = np.bincount(slot, minlength=count) * 39 * 2 * 20 * 2.0 ** -24 * np.abs(g).max()
    assert (np.abs(gl.cpu().numpy() - want) <= bound + 1e-6 * np.abs(want)).all()


@pytest.mark.parametrize("shape,K", [((70, 12, 12), 2), ((5, 20, 24), 1), ((800, 30, 30), 2), ((9, 40, 56), 2), ((900, 64, 64), 1)])
def test_a_lambda_a_plane(shape, K):
    """The same gradient, bit for bit, as with one lambda more, which no plane uses."""
    from gpuutil import run_2d
    rng = np.random.default_rng(shape[0])
    y, g = (rng.normal(size=shape).astype(np.float32) for _ in range(2))
    lam = (10 ** rng.uniform(-2, 0, size=shape[0] + 1)).astype(np.float32)
    own, more = run_2d(y, lam[:-1], K, g), run_2d(y, lam, K, g)
    assert np.array_equal(own["gl"], more["gl"][:-1]) and more["gl"][-1] == 0
    assert np.array_equal(own["gy"], more["gy"])
