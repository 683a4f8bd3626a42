"""Rows that start on no 16-byte boundary move in 16-byte pieces all the same: same bits as from a boundary, and
nothing written outside the rows."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 64, 97, 128, 258, 512, 515, 771, 1027, 3001, 8191, 16382])
def test_same_bits_from_any_float(n):
    import torch

    import paper_2204_03643_amd as tv

    R, dev = 5, torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(n)
    y0 = torch.randn(R, n, generator=gen, device=dev)
    y0[::2] = y0[::2].mul(0.1).cumsum(-1)
    g0 = torch.randn(R, n, generator=gen, device=dev)
    lam = torch.rand(R, generator=gen, device=dev)
    rows, L = tv.rows_along((R, n), -1), tv.tv_lambda(lam.data_ptr(), R, 1)
    wsb = tv.tv1d_bwd_workspace_bytes(rows, L)
    ws = torch.empty(max(16, wsb), dtype=torch.uint8, device=dev)
    first = None
    for off in range(4):
        def place(t):
            room = torch.full((R * n + 8,), float("nan"), device=dev)
            if t is not None:
                room[off:off + R * n] = t.reshape(-1)
            return room, room[off:off + R * n]
        (_, y), (xr, x), (_, g), (gr, gy) = place(y0), place(None), place(g0), place(None)
        gl = torch.empty_like(lam)
        tv.tv1d_prox_fwd(y, x, rows, L)
        tv.tv1d_prox_bwd(g, x, gy, gl, rows, L, ws, wsb)
        for room in (xr, gr):
            assert torch.isnan(room[:off]).all() and torch.isnan(room[off + R * n:]).all(), off
        now = (x.clone(), gy.clone(), gl)
        assert all(torch.isfinite(t).all() for t in now)
        if first is None:
            first = now
        assert all(torch.equal(a, b) for a, b in zip(first, now)), off
