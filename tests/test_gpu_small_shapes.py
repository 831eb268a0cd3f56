"""Launch shapes at their edges, against the oracle: work split finely because a layer is small, tiles that a layer
fills only partly, remainders on both sides of a tile."""
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_1606_04487_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1606_04487_amd import binding
    assert torch.cuda.is_available()
    return binding


def gpu(a, dtype=0):
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return t.to(torch.bfloat16) if dtype == 1 else t


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def rel(got, ref):
    return np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30)


# few channels and images: window rows over workgroups, groups of one image, narrow bands; ragged columns
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("cfg", [(1, 1, 7, 9, 3, 1, 1), (3, 2, 32, 32, 5, 1, 2), (5, 3, 31, 29, 5, 1, 2), (2, 1, 227, 225, 11, 4, 0),
                                 (1, 3, 230, 100, 3, 1, 1), (33, 3, 16, 15, 4, 2, 1), (70, 40, 8, 8, 1, 1, 0)])
def test_lowering_of_small_layers_is_exact(B, cfg, dtype):
    N, C, H, W, k, s, p = cfg
    rng = np.random.default_rng(5)
    X = wl.to_bf16_values(rng.standard_normal((N, C, H, W)))
    d = B.conv_desc(N, C, H, W, 8, k, k, s, p, dtype)
    ld = B.conv_dhat_ld(d)
    D = host(B.lower(d, gpu(X, dtype), None, ld))
    sh = oracle.shape(N, C, H, W, 8, k, k, s, p)
    ref = oracle.lower(sh, X)
    assert np.array_equal(D[:, :ref.shape[1]], ref)
    assert not D[:, ref.shape[1]:].any()


# whole-image windows: D-hat and dY-hat are transposes; images around the 256 rows of a round, odd features
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("N,C,hw,F", [(1, 3, 1, 5), (63, 37, 1, 33), (255, 5, 3, 40), (256, 64, 2, 130), (257, 33, 1, 64), (600, 9, 1, 7)])
def test_fully_connected_layers_of_odd_sizes(B, N, C, hw, F, dtype):
    rng = np.random.default_rng(N)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    X, W = val(rng.standard_normal((N, C, hw, hw))), val(0.05 * rng.standard_normal((F, C, hw, hw)))
    dY = val(rng.standard_normal((N, F, 1, 1)))
    s = oracle.shape(N, C, hw, hw, F, hw, hw, 1, 0)
    tol = 2e-2 if dtype == 1 else 1e-4
    for flags in (0, B.FLAG_SPLIT_K):
        d = B.conv_desc(N, C, hw, hw, F, hw, hw, 1, 0, dtype, flags)
        ws = torch.empty(max(B.conv_workspace_bytes(d, B.PASS_FORWARD), B.conv_workspace_bytes(d, B.PASS_BACKWARD_WEIGHTS)),
                         dtype=torch.uint8, device="cuda")
        Y = B.conv_forward(d, gpu(X, dtype), gpu(W, dtype), None, workspace=ws)
        assert rel(host(Y), oracle.conv_forward(s, X, W, None)) <= tol
        dW, db = B.conv_backward_weights(d.with_flags(flags | B.FLAG_DHAT_CACHED), None, gpu(dY, dtype), workspace=ws)
        assert rel(host(dW), oracle.conv_backward_weights(s, X, dY)) <= 1e-4
        assert rel(host(db), oracle.bias_grad(s, dY)) <= 1e-4


# result rows and columns around the edges of every tile of the lowered products (32 ... 256 rows, 64 ... 256 columns),
# reductions shorter than a step and over several; many images make the model gradient's reduction deep and narrow
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("cfg", [(1, 1, 5, 5, 31, 1, 0), (2, 3, 9, 8, 33, 3, 1), (40, 3, 20, 20, 32, 5, 2), (9, 7, 16, 15, 65, 3, 1),
                                 (3, 16, 24, 24, 96, 3, 0), (7, 20, 13, 13, 193, 2, 0), (13, 48, 14, 14, 257, 3, 1),
                                 (64, 3, 32, 32, 8, 5, 2)])
def test_lowered_products_at_tile_edges(B, cfg, dtype):
    N, C, H, W, F, k, p = cfg
    rng = np.random.default_rng(F)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    X, Wt = val(rng.standard_normal((N, C, H, W))), val(0.05 * rng.standard_normal((F, C, k, k)))
    s = oracle.shape(N, C, H, W, F, k, k, 1, p)
    ho, wo = oracle.out_dims(s)
    dY, b = val(rng.standard_normal((N, F, ho, wo))), (0.05 * rng.standard_normal(F)).astype(np.float32)
    tol = 2e-2 if dtype == 1 else 1e-4
    d = B.conv_desc(N, C, H, W, F, k, k, 1, p, dtype)
    assert rel(host(B.conv_forward(d, gpu(X, dtype), gpu(Wt, dtype), gpu(b))), oracle.conv_forward(s, X, Wt, b)) <= tol
    assert rel(host(B.conv_backward_data(d, gpu(dY, dtype), gpu(Wt, dtype))), oracle.conv_backward_data(s, dY, Wt)) <= tol
    dW, db = B.conv_backward_weights(d, gpu(X, dtype), gpu(dY, dtype))
    assert rel(host(dW), oracle.conv_backward_weights(s, X, dY)) <= 1e-4
    assert rel(host(db), oracle.bias_grad(s, dY)) <= 1e-4


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("tile", range(8))
def test_every_product_tile(B, tile, dtype):
    N, C, H, F, k, p = 5, 24, 17, 200, 3, 1
    rng = np.random.default_rng(tile)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    X, Wt = val(rng.standard_normal((N, C, H, H))), val(0.05 * rng.standard_normal((F, C, k, k)))
    dY = val(rng.standard_normal((N, F, H, H)))
    s = oracle.shape(N, C, H, H, F, k, k, 1, p)
    tol = 2e-2 if dtype == 1 else 1e-4
    d = B.conv_desc(N, C, H, H, F, k, k, 1, p, dtype)
    B.tuning_set(B.TUNE_GEMM_TILE, tile)
    try:
        assert rel(host(B.conv_forward(d, gpu(X, dtype), gpu(Wt, dtype), None)), oracle.conv_forward(s, X, Wt, None)) <= tol
        assert rel(host(B.conv_backward_data(d, gpu(dY, dtype), gpu(Wt, dtype))), oracle.conv_backward_data(s, dY, Wt)) <= tol
        assert rel(host(B.conv_backward_weights(d, gpu(X, dtype), gpu(dY, dtype))[0]), oracle.conv_backward_weights(s, X, dY)) <= 1e-4
    finally:
        B.tuning_set(B.TUNE_GEMM_TILE, -1)


# One or two steps of loads in flight, by the length of the reduction (up to five steps: one): every tile of the lowered products
# over 4 to 9 steps, whole and ending inside the last one.  A window of 1 x 1: the forward pass reduces over the channels, the data
# gradient over the filters.
@functools.lru_cache(maxsize=None)
def one_by_one(channels, dtype):
    N, H, W = 3, 11, 13
    rng = np.random.default_rng(channels)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    X, Wt = val(rng.standard_normal((N, channels, H, W))), val(0.05 * rng.standard_normal((channels, channels, 1, 1)))
    s = oracle.shape(N, channels, H, W, channels, 1, 1, 1, 0)
    return X, Wt, oracle.conv_forward(s, X, Wt, None), oracle.conv_backward_data(s, X, Wt)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("tile", range(8))
@pytest.mark.parametrize("steps,less", [(4, 0), (5, 3), (5, 0), (6, 13), (6, 0), (7, 1), (8, 0), (9, 16)])
def test_steps_in_flight(B, steps, less, tile, dtype):
    channels = steps * (64 if dtype == 1 else 32) - less
    X, Wt, Y, dX = one_by_one(channels, dtype)
    d = B.conv_desc(X.shape[0], channels, X.shape[2], X.shape[3], channels, 1, 1, 1, 0, dtype)
    # one rounding to bf16, and fp32 sums of up to 576 products
    close = lambda got, ref: np.all(np.abs(got - ref) <= (2.0 ** -8 if dtype == 1 else 0.0) * np.abs(ref) + 1e-5 * np.max(np.abs(ref)))
    B.tuning_set(B.TUNE_GEMM_TILE, tile)
    B.tuning_set(B.TUNE_DGRAD_CONV, 1)
    try:
        assert close(host(B.conv_forward(d, gpu(X, dtype), gpu(Wt, dtype), None)), Y)
        assert close(host(B.conv_backward_data(d, gpu(X, dtype), gpu(Wt, dtype))), dX)
    finally:
        B.tuning_set(B.TUNE_GEMM_TILE, -1)
        B.tuning_set(B.TUNE_DGRAD_CONV, 0)


# reductions split over the chip, of 8 to 40 steps: last ranges of one step to a whole range, which the same launch runs
@pytest.mark.parametrize("dtype", [0, 1])
def test_last_ranges_of_split_products(B, dtype):
    N, F, step = 70, 40, 64 if dtype == 1 else 32
    rng = np.random.default_rng(3)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    for steps in range(8, 41):
        C = step * steps - steps % 3
        X, Wt = val(rng.standard_normal((N, C, 1, 1))), val(0.05 * rng.standard_normal((F, C, 1, 1)))
        d = B.conv_desc(N, C, 1, 1, F, 1, 1, 1, 0, dtype, B.FLAG_SPLIT_K)
        ref = (X.reshape(N, C).astype(np.float64) @ Wt.reshape(F, C).astype(np.float64).T)
        got = host(B.conv_forward(d, gpu(X, dtype), gpu(Wt, dtype), None)).reshape(N, F)
        assert np.all(np.abs(got - ref) <= (2.0 ** -8 if dtype == 1 else 0.0) * np.abs(ref) + 1e-5 * np.max(np.abs(ref))), steps
        back = B.conv_desc(N, F, 1, 1, C, 1, 1, 1, 0, dtype, B.FLAG_SPLIT_K)      # the filters of this layer are the reduction
        ref = (X.reshape(N, C).astype(np.float64) @ Wt.reshape(F, C).astype(np.float64).T)
        got = host(B.conv_backward_data(back, gpu(X, dtype), gpu(np.ascontiguousarray(Wt.reshape(F, C).T).reshape(C, F, 1, 1), dtype))).reshape(N, F)
        assert np.all(np.abs(got - ref) <= (2.0 ** -8 if dtype == 1 else 0.0) * np.abs(ref) + 1e-5 * np.max(np.abs(ref))), steps


# split reductions of the fused convolution: one and four results per thread of the summing launch, pieces that straddle
# images and filters (odd planes), split counts below, at and above the eight loads in flight
@pytest.mark.parametrize("N,C,HW,F", [(3, 64, 9, 37), (9, 64, 15, 200), (5, 256, 13, 384), (5, 288, 13, 384), (1, 384, 7, 130)])
def test_sums_of_split_fused_products(B, N, C, HW, F):
    rng = np.random.default_rng(C + F)
    X, Wt = wl.to_bf16_values(rng.standard_normal((N, C, HW, HW))), wl.to_bf16_values(0.05 * rng.standard_normal((F, C, 3, 3)))
    b = (0.05 * rng.standard_normal(F)).astype(np.float32)
    s = oracle.shape(N, C, HW, HW, F, 3, 3, 1, 1)
    d = B.conv_desc(N, C, HW, HW, F, 3, 3, 1, 1, 1, B.FLAG_FUSED | B.FLAG_RELU)
    assert B.conv_fused_supported(d, B.PASS_FORWARD)
    Y = host(B.conv_forward(d, gpu(X, 1), gpu(Wt, 1), gpu(b)))
    ref = np.maximum(oracle.conv_forward(s, X, Wt, b), 0.0)
    # one rounding to bf16, and fp32 sums
    assert np.all(np.abs(Y - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-4 * np.max(np.abs(ref)))


# the fused convolution's 64 x 128 tile: filters and columns around a tile's edges, tiles over several images, split and
# whole reductions, one to eight images per tile, a conflict-free pitch and (27 x 27, window 5) a bare one
@pytest.mark.parametrize("N,C,H,W,F,k,p", [(1, 32, 9, 14, 63, 3, 1), (1, 32, 16, 8, 64, 3, 1), (1, 64, 3, 43, 65, 3, 1), (7, 96, 5, 5, 129, 3, 1),
                                           (2, 96, 27, 27, 200, 5, 2), (3, 192, 13, 13, 256, 3, 1), (40, 32, 8, 8, 32, 5, 2), (5, 64, 17, 12, 96, 1, 0),
                                           (2, 32, 32, 31, 40, 5, 0), (1, 448, 7, 9, 1, 3, 2)])
def test_small_tile_of_the_fused_convolution(B, N, C, H, W, F, k, p):
    rng = np.random.default_rng(N + F)
    X, Wt = wl.to_bf16_values(rng.standard_normal((N, C, H, W))), wl.to_bf16_values(0.05 * rng.standard_normal((F, C, k, k)))
    b = (0.05 * rng.standard_normal(F)).astype(np.float32)
    s = oracle.shape(N, C, H, W, F, k, k, 1, p)
    ho, wo = oracle.out_dims(s)
    dY = wl.to_bf16_values(rng.standard_normal((N, F, ho, wo)))
    d = B.conv_desc(N, C, H, W, F, k, k, 1, p, 1, B.FLAG_FUSED)
    close = lambda got, ref: np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-4 * np.max(np.abs(ref)))  # one rounding, fp32 sums
    B.tuning_set(B.TUNE_FUSED_BN, 128)
    try:
        assert B.conv_fused_supported(d, B.PASS_FORWARD)
        assert close(host(B.conv_forward(d, gpu(X, 1), gpu(Wt, 1), gpu(b))), oracle.conv_forward(s, X, Wt, b))
        if B.conv_fused_supported(d, B.PASS_BACKWARD_DATA):
            assert close(host(B.conv_backward_data(d, gpu(dY, 1), gpu(Wt, 1))), oracle.conv_backward_data(s, dY, Wt))
    finally:
        B.tuning_set(B.TUNE_FUSED_BN, 0)


# its masked, row-form output: the same results as the tile the library chooses
@pytest.mark.parametrize("N,C,H,F", [(392, 64, 13, 128), (392, 192, 13, 128)])
def test_small_tile_behind_a_relu_mask(B, N, C, H, F):
    rng = np.random.default_rng(C)
    bf = lambda a: gpu(a, 1)
    Wt, dY = bf(0.05 * rng.standard_normal((F, C, 3, 3))), bf(rng.standard_normal((N, F, H, H)))
    y_front = bf(np.maximum(rng.standard_normal((N, C, H, H)), 0.0))
    d = B.conv_desc(N, C, H, H, F, 3, 3, (1, 1), (1, 1), 1, B.FLAG_FUSED)
    packed = torch.empty(B.conv_packed_weights_bytes(d, B.PASS_BACKWARD_DATA), dtype=torch.uint8, device="cuda")
    B.conv_pack_weights([d], [B.PASS_BACKWARD_DATA], [Wt], [packed])
    pitch = (H * H + 7) // 8 * 8
    rows = torch.zeros((F, N, pitch), dtype=torch.bfloat16, device="cuda")
    rows[:, :, :H * H] = dY.reshape(N, F, H * H).transpose(0, 1)
    rows = rows.reshape(F, N * pitch)
    expect = B.conv_backward_data_rows(d, rows, packed).float() * (y_front > 0)
    B.tuning_set(B.TUNE_FUSED_BN, 128)
    try:
        got, sums = B.conv_backward_data_relu_rows(d, rows, packed, y_front)
    finally:
        B.tuning_set(B.TUNE_FUSED_BN, 0)
    planes = got.float().reshape(C, N, pitch)[:, :, :H * H].transpose(0, 1).reshape(N, C, H, H)
    assert torch.equal(planes, expect)   # the order of a result's terms does not depend on the tile
    total = host(expect).sum(axis=(0, 2, 3))
    assert np.max(np.abs(host(sums).sum(axis=1) - total)) <= 1e-5 * np.max(np.abs(host(expect)).sum(axis=(0, 2, 3)))


# fp32 data gradients by one product over dY, on each of its tiles: channels around the row tiles, columns that fill none,
# filters padded to a step (31, 33, 40, 70) or not, one to eight steps per tap and more (257), windows that reach beyond
# the border on all sides, planes narrower than a wavefront, windows of 1 and of 31 taps.  The terms and their order are
# those of the route over dD-hat: the same bits.
@pytest.mark.parametrize("tile", [0, 3, 4, 5, 6])
@pytest.mark.parametrize("N,C,H,W,F,k,p", [(2, 33, 9, 14, 31, 3, 1), (9, 96, 27, 27, 64, 5, 2), (3, 64, 16, 16, 33, 5, 2), (40, 32, 8, 8, 256, 5, 2),
                                           (2, 130, 20, 23, 70, 3, 0), (64, 65, 7, 7, 40, 3, 2), (5, 200, 13, 13, 257, 1, 0), (16, 129, 31, 31, 8, 3, 1),
                                           (3, 5, 33, 6, 40, (31, 1), (30, 0))])
def test_fp32_data_gradient_by_one_product(B, N, C, H, W, F, k, p, tile):
    rng = np.random.default_rng(C)
    (kh, kw), (ph, pw) = k if isinstance(k, tuple) else (k, k), p if isinstance(p, tuple) else (p, p)
    Wt = (0.05 * rng.standard_normal((F, C, kh, kw))).astype(np.float32)
    s = oracle.shape(N, C, H, W, F, kh, kw, 1, (ph, pw))
    dY = rng.standard_normal((N, F) + tuple(oracle.out_dims(s))).astype(np.float32)
    d = B.conv_desc(N, C, H, W, F, kh, kw, 1, (ph, pw), 0)
    ref = oracle.conv_backward_data(s, dY, Wt)
    dYg, Wg = gpu(dY), gpu(Wt)

    def run(route):
        B.tuning_set(B.TUNE_DGRAD_CONV, route)
        try:
            return B.conv_backward_data(d, dYg, Wg)
        finally:
            B.tuning_set(B.TUNE_DGRAD_CONV, 0)
    lowered, here = run(1), run(2 + tile)
    assert rel(host(here), ref) <= 2e-6   # sums of a few hundred products and of those: some 1e-7 of the tensor's scale
    assert torch.equal(here, lowered)
    # an infinite entry behind the last channel of an image: no other image's gradient may see it
    dYg[1, 0] = float("inf")
    bad, keep = run(2 + tile), [n for n in range(N) if n != 1]
    assert torch.equal(bad[keep], here[keep])
    assert torch.equal(torch.nan_to_num(bad, 7.0, 8.0, 9.0), torch.nan_to_num(run(1), 7.0, 8.0, 9.0))


# an image's data gradient does not depend on the batch it is computed in, whichever route the batch's size selects
@pytest.mark.parametrize("C,H,F,k,p", [(32, 16, 32, 5, 2), (96, 27, 256, 5, 2), (256, 13, 384, 3, 1)])
def test_fp32_data_gradient_does_not_depend_on_the_batch(B, C, H, F, k, p):
    g = torch.Generator(device="cuda").manual_seed(k)
    Wt = 0.05 * torch.randn((F, C, k, k), device="cuda", generator=g)
    dY = torch.randn((128, F, H, H), device="cuda", generator=g)
    full = B.conv_backward_data(B.conv_desc(128, C, H, H, F, k, k, 1, p, 0), dY, Wt)
    for n in (1, 7, 48):
        part = B.conv_backward_data(B.conv_desc(n, C, H, H, F, k, k, 1, p, 0), dY[:n].contiguous(), Wt)
        assert torch.equal(part, full[:n])


# weights that are infinite or NaN in one tap: only input pixels that this tap joins to an output position see them, on
# every tile of the in-place product as on the route over dD-hat
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("N,C,H,F,k,p", [(3, 33, 9, 31, 3, 1), (2, 40, 7, 64, 5, 2), (2, 40, 8, 33, 3, 0)])
def test_fp32_data_gradient_of_weights_that_are_not_finite(B, N, C, H, F, k, p, value):
    g = torch.Generator(device="cuda").manual_seed(k)
    Ho = H + 2 * p - k + 1
    Wt = 0.05 * torch.randn((F, C, k, k), device="cuda", generator=g)
    dY = torch.randn((N, F, Ho, Ho), device="cuda", generator=g)
    d = B.conv_desc(N, C, H, H, F, k, k, 1, p, 0)
    clean = B.conv_backward_data(d, dY, Wt)
    Wt[:, :, 0, k - 1] = value
    joined = torch.zeros((H, H), dtype=torch.bool, device="cuda")   # pixel (y, x) meets tap (0, k - 1) at (y + p, x + p - k + 1)
    joined[max(0, -p):Ho - p, max(0, k - 1 - p):Ho - p + k - 1] = True
    for route in (1, 2, 5, 6, 7, 8):
        B.tuning_set(B.TUNE_DGRAD_CONV, route)
        try:
            got = B.conv_backward_data(d, dY, Wt)
        finally:
            B.tuning_set(B.TUNE_DGRAD_CONV, 0)
        assert not torch.isfinite(got[:, :, joined]).any()
        assert torch.isfinite(got[:, :, ~joined]).all()
        kept = torch.allclose(got[:, :, ~joined], clean[:, :, ~joined], rtol=0, atol=0)
        assert kept, route


# split products on each of their tiles: rows of 32, 64 and 128, columns of 64 and 128, results that pad them, forward and
# (whole-image window) data gradient
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("N,K,F", [(3, 1088, 640), (32, 2048, 512), (33, 1024, 1088), (64, 4160, 512), (65, 1024, 1160), (130, 2112, 2112), (256, 8200, 512)])
def test_split_products_of_fully_connected_layers(B, N, K, F, dtype):
    rng = np.random.default_rng(N)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    X, W = val(rng.standard_normal((N, K, 1, 1))), val(0.05 * rng.standard_normal((F, K, 1, 1)))
    dY, b = val(rng.standard_normal((N, F, 1, 1))), (0.05 * rng.standard_normal(F)).astype(np.float32)
    d = B.conv_desc(N, K, 1, 1, F, 1, 1, 1, 0, dtype, B.FLAG_SPLIT_K)
    Xd, Wd, dYd = (a.astype(np.float64).reshape(a.shape[:2]) for a in (X, W, dY))
    # one rounding to bf16, and fp32 sums
    close = lambda got, ref: np.all(np.abs(got.reshape(ref.shape) - ref) <= (2.0 ** -8 if dtype == 1 else 0.0) * np.abs(ref) + 1e-5 * np.max(np.abs(ref)))
    assert close(host(B.conv_forward(d, gpu(X, dtype), gpu(W, dtype), gpu(b))), Xd @ Wd.T + b.astype(np.float64))
    assert close(host(B.conv_backward_data(d, gpu(dY, dtype), gpu(W, dtype))), dYd @ Wd)


# the same data gradient with F no multiple of a reduction step (64 in bf16, 32 in fp32): the last step ends inside an image's
# row of dY, and what follows there -- the next image's row, infinite here -- belongs to no sum of this one
@pytest.mark.parametrize("flags", [0, 8])   # SPLIT_K
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("N,K,F", [(3, 256, 8), (16, 4096, 1000), (33, 1024, 1000), (64, 512, 72), (130, 2048, 1048), (300, 4096, 1000), (600, 1024, 24)])
def test_dense_data_gradient_whose_reduction_ends_inside_a_step(B, N, K, F, dtype, flags):
    rng = np.random.default_rng(N)
    val = wl.to_bf16_values if dtype == 1 else (lambda a: a.astype(np.float32))
    W, dY = val(0.05 * rng.standard_normal((F, K, 1, 1))), val(rng.standard_normal((N, F, 1, 1)))
    d = B.conv_desc(N, K, 1, 1, F, 1, 1, 1, 0, dtype, flags)
    ref = dY.astype(np.float64).reshape(N, F) @ W.astype(np.float64).reshape(F, K)
    dYg, Wg = gpu(dY, dtype), gpu(W, dtype)
    got = B.conv_backward_data(d, dYg, Wg)
    # one rounding to bf16, and fp32 sums
    assert np.all(np.abs(host(got).reshape(N, K) - ref) <= (2.0 ** -8 if dtype == 1 else 0.0) * np.abs(ref) + 1e-5 * np.max(np.abs(ref)))
    dYg[1::2] = float("inf")
    assert torch.equal(B.conv_backward_data(d, dYg, Wg)[0::2], got[0::2])


# model gradient of the 13 x 13 layers over one image range (one image, or forced): the product stores the gradient itself
@pytest.mark.parametrize("N,splits", [(1, 0), (3, 1)])
def test_model_gradient_without_partial_sums(B, N, splits):
    C, F, H = 64, 128, 13
    rng = np.random.default_rng(N)
    X, dY = wl.to_bf16_values(rng.standard_normal((N, C, H, H))), wl.to_bf16_values(rng.standard_normal((N, F, H, H)))
    s = oracle.shape(N, C, H, H, F, 3, 3, 1, 1)
    d = B.conv_desc(N, C, H, H, F, 3, 3, 1, 1, 1, B.FLAG_FUSED)
    ref, ref_b = oracle.conv_backward_weights(s, X, dY), oracle.bias_grad(s, dY)
    B.tuning_set(B.TUNE_WGRAD_SPLITS, splits)
    try:
        dW, db = B.conv_backward_weights(d, gpu(X, 1), gpu(dY, 1))
    finally:
        B.tuning_set(B.TUNE_WGRAD_SPLITS, 0)
    assert rel(host(dW), ref) <= 1e-4 and rel(host(db), ref_b) <= 1e-4


# A split product's error against 64 bits: a chain of L fp32 terms leaves about 0.3 x 2^-24 sqrt(L) of the result's norm
# (measured over L from 256 to 30 000).  Ranges are never fewer, chains never longer than one workgroup per compute unit
# on 256 x 256 tiles or two on 128 x 128 give: 128 x 576 over 802 816 has 102 ranges, 256 x 4096 over 4096 has 16.
def test_error_of_split_products_against_64_bits(B):
    g = torch.Generator(device="cuda").manual_seed(3)
    err = lambda got, ref: float((got.double().reshape(ref.shape) - ref).norm() / ref.norm())
    limit = lambda chain: 0.4 * 2.0 ** -24 * chain ** 0.5
    N, C, F, hw = 64, 576, 128, 112 * 112
    X, dY = torch.randn((N, C, 112, 112), device="cuda", generator=g), torch.randn((N, F, 112, 112), device="cuda", generator=g)
    dW, _ = B.conv_backward_weights(B.conv_desc(N, C, 112, 112, F, 1, 1, 1, 0, 0), X, dY)
    ref = sum(dY[n].reshape(F, hw).double() @ X[n].reshape(C, hw).double().t().contiguous() for n in range(N))
    assert err(dW, ref) <= limit(N * hw / 102)
    del X, dY
    X, W = torch.randn((256, 4096, 1, 1), device="cuda", generator=g), torch.randn((4096, 4096, 1, 1), device="cuda", generator=g)
    d = B.conv_desc(256, 4096, 1, 1, 4096, 1, 1, 1, 0, 0, B.FLAG_SPLIT_K)
    Xd, Wd = X.reshape(256, 4096).double(), W.reshape(4096, 4096).double()
    assert err(B.conv_forward(d, X, W), Xd @ Wd.t().contiguous()) <= limit(4096 / 16)
    assert err(B.conv_backward_data(d, X, W), Xd @ Wd) <= limit(4096 / 16)


# the profile's records: preparations that share a launch count under its class with the bytes of both, and no launch twice
@pytest.mark.parametrize("dtype", [0, 1])
def test_profile_of_preparations_that_share_a_launch(B, dtype):
    N, C, H, F, k, e = 4, 8, 12, 24, 3, 4 if dtype == 0 else 2
    M, K = N * H * H, C * k * k
    d = B.conv_desc(N, C, H, H, F, k, k, 1, 1, dtype)
    g = torch.Generator(device="cuda").manual_seed(1)
    mk = lambda *s: torch.randn(s, device="cuda", generator=g).to(B.torch_dtype(dtype))
    X, W, dY = mk(N, C, H, H), mk(F, C, k, k), mk(N, F, H, H)
    fc = B.conv_desc(20, 40, 1, 1, 48, 1, 1, 1, 0, dtype)
    fX, fdY = mk(20, 40, 1, 1), mk(20, 48, 1, 1)

    def records(call):
        B.profile_enable(True)
        try:
            call()
            return {n: (r["launches"], r["bytes"]) for n, r in B.profile_summary().items() if r["launches"] and r["bytes"]}
        finally:
            B.profile_enable(False)
    x, w, dhat, dy = N * C * H * H * e, F * K * e, K * M * e, F * M * e
    fwd = records(lambda: B.conv_forward(d, X, W))
    assert fwd["lower"] == (1, x + dhat + 2 * w) and "pack_khat" not in fwd
    B.tuning_set(B.TUNE_DGRAD_CONV, 1)
    try:
        bwd = records(lambda: B.conv_backward_data(d, dY, W))
    finally:
        B.tuning_set(B.TUNE_DGRAD_CONV, 0)
    assert bwd["pack_dyhat"] == (1, 2 * dy + 2 * w) and "pack_khat" not in bwd
    wgr = records(lambda: B.conv_backward_weights(d, X, dY))
    assert wgr["lower"] == (1, x + dhat + 2 * dy) and "pack_dyhat" not in wgr
    fcw = records(lambda: B.conv_backward_weights(fc, fX, fdY))
    assert fcw["pack_dyhat"] == (1, 2 * 20 * 48 * e) and fcw["lower"] == (1, 2 * 20 * 40 * e) and "bias_reduce" not in fcw
