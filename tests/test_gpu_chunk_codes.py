"""2D calls on sides of 65-768 samples leave chunk codes for the reverse sweep instead of pass outputs."""
import numpy as np
import pytest

from gpuutil import run_2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,K,count", [
    (65, 96, 1, 2), (97, 65, 2, 3), (128, 97, 3, 1), (129, 192, 2, 2), (256, 193, 1, 1), (193, 257, 4, 3),
    (384, 385, 3, 1), (512, 512, 2, 2), (321, 481, 3, 3), (513, 768, 3, 1), (768, 513, 1, 3), (768, 65, 2, 1)])
def test_codes_and_kept_passes_give_the_same_bits(H, W, K, count):
    """Both ends of every thread mapping, rows and columns, block means and elimination (one lambda,
    three sweeps), cold and warm passes: x, grad_y and grad_lam are bit for bit what the call gives when
    it keeps its pass outputs, the reverse sweep telling the two apart by the workspace alone."""
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(H * 1000 + W)
    y = (np.cumsum(rng.normal(scale=0.05, size=(3, H, W)), axis=-1) + rng.normal(scale=0.2, size=(3, H, W))).astype(np.float32)
    y[1] = np.maximum(y[1], 0)                                  # ties
    y[2, 5, 7:9] = np.inf                                       # equal infinities are no jump
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = (10 ** rng.uniform(-2, 0, size=count)).astype(np.float32)
    kept = run_2d(y, lam, K, g, keep_passes=True)
    bytes_ = tv.tv_dispatch_threshold("chunk_codes_bytes")
    tv.tv_dispatch_override("chunk_codes_bytes", 0)
    try:
        lean = run_2d(y, lam, K, g, keep_passes=False)
    finally:
        tv.tv_dispatch_override("chunk_codes_bytes", bytes_)
    for k in ("x", "gy", "gl"):
        assert np.array_equal(kept[k], lean[k], equal_nan=True), k
    assert np.array_equal(kept["saved"][2 * K - 1], kept["x"], equal_nan=True)


@pytest.mark.parametrize("H,W,K,count", [(65, 96, 1, 2), (96, 70, 2, 3), (97, 65, 2, 3), (128, 97, 3, 1), (129, 192, 2, 2), (192, 66, 1, 3), (256, 193, 1, 1)])
def test_codes_read_by_the_columns_of_a_large_call(H, W, K, count):
    """The same with the mappings that more than "bwd_few_columns" columns have, whose threads read a word or two each where
    those of few columns read half a word or one; and the two mappings agree to rounding."""
    import paper_2204_03643_amd as tv
    rng = np.random.default_rng(H * 1000 + W)
    y = (np.cumsum(rng.normal(scale=0.05, size=(3, H, W)), axis=-2) + rng.normal(scale=0.2, size=(3, H, W))).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = (10 ** rng.uniform(-2, 0, size=count)).astype(np.float32)
    saved = {k: tv.tv_dispatch_threshold(k) for k in ("chunk_codes_bytes", "bwd_few_columns")}
    try:
        tv.tv_dispatch_override("chunk_codes_bytes", 0)
        few = run_2d(y, lam, K, g, keep_passes=False)
        tv.tv_dispatch_override("bwd_few_columns", 0)
        lean = run_2d(y, lam, K, g, keep_passes=False)
        kept = run_2d(y, lam, K, g, keep_passes=True)
    finally:
        for k, v in saved.items():
            tv.tv_dispatch_override(k, v)
    for k in ("x", "gy", "gl"):
        assert np.array_equal(kept[k], lean[k]), k
    # sums of 64 bits over other chunks: a mean may round the other way in each of the 2 K passes; and the floats that threads
    # leave of dL/dlam, at most 16 a column of two means each, in each of the K column passes
    largest = max(np.abs(g).max(), np.abs(few["gy"]).max())
    assert np.abs(few["gy"] - lean["gy"]).max() <= 2 * K * 2.0 ** -23 * largest
    assert np.abs(few["gl"] - lean["gl"]).max() <= 2.0 ** -23 * (K * 3 * W * 16 * 2 * largest + np.abs(few["gl"]).max())


def test_reverse_sweep_twice_on_one_workspace():
    """The reverse sweep only reads the codes: a second one on the same workspace gives the same bits
    (63 lambdas: the reduction split over the most workgroups it has, beside the word that tells
    codes from pass outputs)."""
    import torch

    import paper_2204_03643_amd as tv
    planes, H, W, K = 63, 66, 70, 40
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    y, g = (torch.randn((planes, H, W), generator=gen, device="cuda") for _ in range(2))
    lam = torch.full((planes,), 0.2, device="cuda")
    L = tv.tv_lambda(lam.data_ptr(), planes, 1)
    wsb = tv.tv2d_workspace_bytes(planes, H, W, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    x = torch.empty_like(y)
    tv.tv2d_prox_fwd(y, x, planes, H, W, L, K, ws, wsb)
    out = []
    for _ in range(2):
        gy, gl = torch.empty_like(y), torch.empty_like(lam)
        tv.tv2d_prox_bwd(g, gy, gl, planes, H, W, L, K, ws, wsb)
        out.append((gy, gl))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert bool(torch.isfinite(out[0][0]).all())


@pytest.fixture
def overrides():
    import paper_2204_03643_amd as tv
    saved = {}

    def set_to(**values):
        for name, value in values.items():
            saved.setdefault(name, tv.tv_dispatch_threshold(name))
            tv.tv_dispatch_override(name, value)
    yield set_to
    for name, value in saved.items():
        tv.tv_dispatch_override(name, value)


def _kept_and_codes(y, lam, K, g, overrides):
    """The call with its pass outputs kept, and with codes in their place."""
    kept = run_2d(y, lam, K, g, keep_passes=True)
    overrides(chunk_codes_bytes=0)
    return kept, run_2d(y, lam, K, g, keep_passes=False)


@pytest.mark.parametrize("H,W,K,count", [(65, 97, 3, 1), (130, 96, 3, 1), (200, 260, 3, 1), (400, 70, 3, 1), (65, 97, 2, 3), (300, 130, 1, 1)])
@pytest.mark.parametrize("value", [0.0, -1.0])
def test_zeros_of_both_signs_are_no_jump(H, W, K, count, value, overrides):
    """lambda = 0 leaves a masked image as it is, zeros of both signs included: no code may call -0 beside
    +0 a jump, by elimination (one lambda, three sweeps) or by block means."""
    rng = np.random.default_rng(H + W)
    y = rng.normal(size=(3, H, W)).astype(np.float32)
    y = np.where(np.abs(y) < 0.8, np.where(rng.random(y.shape) < 0.5, np.float32(0), np.float32(-0.0)), y).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    kept, lean = _kept_and_codes(y, np.full(count, value, np.float32), K, g, overrides)
    assert np.array_equal(kept["x"], y)
    for k in ("x", "gy", "gl"):
        assert np.array_equal(kept[k], lean[k]), k


@pytest.mark.parametrize("H,W,K,count", [(70, 65, 1, 2), (80, 130, 2, 3), (66, 300, 3, 1), (100, 768, 2, 2)])
@pytest.mark.parametrize("coarsest", [4096, 64])
def test_codes_behind_a_multilevel_first_pass(H, W, K, count, coarsest, overrides):
    """With the multilevel start asked for on these sides, the first pass is several launches, of which the
    last one alone leaves codes and the word that tells codes from pass outputs (one level, and several)."""
    from parity import check_2d
    rng = np.random.default_rng(H + W)
    y = np.cumsum(rng.normal(scale=0.1, size=(3, H, W)), axis=-1).astype(np.float32)
    g = rng.normal(size=y.shape).astype(np.float32)
    lam = (10 ** rng.uniform(-0.5, 0.5, size=count)).astype(np.float32)
    overrides(ml_min_length=65, ml_coarsest=coarsest, one_lambda_tri_side=0)
    kept, lean = _kept_and_codes(y, lam, K, g, overrides)
    check_2d(y, lam, K, g, kept, "multilevel first pass %dx%d" % (H, W))
    for k in ("x", "gy", "gl"):
        assert np.array_equal(kept[k], lean[k]), k


@pytest.mark.parametrize("H,W,K,count", [(65, 97, 2, 3), (192, 130, 3, 1), (260, 384, 1, 2), (513, 768, 2, 3)])
def test_threshold_moved_between_forward_and_reverse(H, W, K, count, overrides):
    """The reverse sweep expects what a forward call leaves at its own moment, and gives the same bits when it
    finds the other."""
    import torch

    import paper_2204_03643_amd as tv
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H)
    y, g = (torch.randn((3, H, W), generator=gen, device="cuda") for _ in range(2))
    lam = torch.full((count,), 0.3, device="cuda")
    L = tv.tv_lambda(lam.data_ptr(), count, 1)
    wsb = tv.tv2d_workspace_bytes(3, H, W, K)
    out = []
    for at_forward in (0, 1 << 40):
        for at_reverse in (0, 1 << 40):
            ws = torch.full((wsb,), 0xff, dtype=torch.uint8, device="cuda")
            x, gy, gl = torch.empty_like(y), torch.empty_like(y), torch.empty_like(lam)
            overrides(chunk_codes_bytes=at_forward)
            tv.tv2d_prox_fwd(y, x, 3, H, W, L, K, ws, wsb)
            overrides(chunk_codes_bytes=at_reverse)
            tv.tv2d_prox_bwd(g, gy, gl, 3, H, W, L, K, ws, wsb)
            out.append((x, gy, gl))
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b)
