"""The fused convolution's small tiles that hold all channels' pixels at once (whole_patch.hip), each of them against the
oracle, and with dY as its rows matrix against the dense call."""
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


@pytest.fixture
def tile(B, request):
    B.tuning_set(B.TUNE_FUSED_WHOLE, 2 + request.param)
    yield request.param
    B.tuning_set(B.TUNE_FUSED_WHOLE, 0)


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


# filters and columns around a tile's edges; planes of odd size (pieces of 7, shifted loads) and of even rows (pieces of 8),
# of 8 and 9 elements, several images per tile; more wavefronts than steps (window 1) and many steps; tiles that lie in the
# padding altogether; patches near the largest that fits
SHAPES = [(1, 32, 2, 4, 5, 1, 0), (3, 32, 3, 3, 33, 3, 1), (1, 32, 8, 8, 32, 1, 3), (7, 64, 5, 5, 63, 3, 1), (2, 96, 27, 27, 70, 5, 2),
          (3, 192, 13, 13, 65, 3, 1), (5, 32, 16, 16, 32, 5, 2), (2, 64, 17, 12, 96, 1, 0), (1, 64, 9, 14, 127, 3, 1), (2, 32, 32, 31, 40, 5, 0),
          (1, 448, 7, 9, 1, 3, 2), (2, 384, 13, 13, 64, 3, 1), (1, 32, 3, 43, 129, 3, 1), (2, 32, 30, 27, 32, 3, 1)]


# (rows, columns) of the tiles, and whether each of a layer's column tiles fits the 158 KB that hold its pixels: a forced tile
# that does not fit is ignored, and a test of it would test the larger tiles
TILES = [(32, 32), (32, 64), (64, 64), (64, 96)]


def fits(tile, N, C, H, W, ho, wo, k, pad):
    rows, columns = TILES[tile]
    most = 0
    for first in range(0, N * ho * wo, columns):
        last = min(first + columns, N * ho * wo) - 1
        images = range(first // (ho * wo), last // (ho * wo) + 1)
        touched = [(max(first - n * ho * wo, 0) // wo, min(last - n * ho * wo, ho * wo - 1) // wo) for n in images]
        if len(touched) > 8:
            return False
        most = max(most, sum(b - a + k for a, b in touched))
    return most * (W + 2 * pad) <= 158 * 1024 // 16 // (C // 8) - 1


@pytest.mark.parametrize("tile", range(4), indirect=True)
@pytest.mark.parametrize("N,C,H,W,F,k,p", SHAPES)
def test_against_the_oracle(B, tile, N, C, H, W, F, k, p):
    print("whole patch", tile, N, C, H, W, F, k, p, flush=True)
    rng = np.random.default_rng(C + F)
    X, Wt = wl.to_bf16_values(rng.standard_normal((N, C, H, W))), wl.to_bf16_values(0.05 * rng.standard_normal((F, C, k, k)))
    b = (0.05 * rng.standard_normal(F)).astype(np.float32)
    s = oracle.shape(N, C, H, W, F, k, k, 1, p)
    ho, wo = oracle.out_dims(s)
    dY = wl.to_bf16_values(rng.standard_normal((N, F, ho, wo)))
    d = B.conv_desc(N, C, H, W, F, k, k, 1, p, 1, B.FLAG_FUSED | B.FLAG_RELU)
    # one rounding to bf16, and fp32 sums
    close = lambda got, ref: np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-4 * np.max(np.abs(ref)))
    Y = torch.full((N, F, ho, wo), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert B.conv_fused_supported(d, B.PASS_FORWARD) and fits(tile, N, C, H, W, ho, wo, k, p)
    B.conv_forward(d, gpu(X), gpu(Wt), torch.from_numpy(b).cuda(), Y)
    assert close(host(Y), np.maximum(oracle.conv_forward(s, X, Wt, b), 0.0))
    if B.conv_fused_supported(d, B.PASS_BACKWARD_DATA):
        assert fits(tile, N, F, ho, wo, H, W, k, k - 1 - p)
        dX = torch.full((N, C, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.conv_backward_data(d, gpu(dY), gpu(Wt), dX)
        assert close(host(dX), oracle.conv_backward_data(s, dY, Wt))


# dY as its rows matrix: pieces that straddle images, a ragged last column tile, channels that fill no row tile, a plane as long as
# its pitch; every stored value is bit-identical to the dense call's.  Behind a ReLU's mask the larger tiles run, whatever is
# forced: their data gradient under that mask, and their column sums.
@pytest.mark.parametrize("tile", range(4), indirect=True)
@pytest.mark.parametrize("N,C,H,W,F,k,p", [(392, 64, 13, 13, 128, 3, 1), (700, 96, 8, 12, 128, 5, 2)])
def test_rows_and_mask(B, tile, N, C, H, W, F, k, p):
    print("whole patch rows", tile, N, C, H, W, F, flush=True)
    rng = np.random.default_rng(N)
    Wt, dY = gpu(0.05 * rng.standard_normal((F, C, k, k))), gpu(rng.standard_normal((N, F, H, W)))
    y_front = gpu(np.maximum(rng.standard_normal((N, C, H, W)), 0.0))
    d = B.conv_desc(N, C, H, W, F, k, k, 1, p, 1, B.FLAG_FUSED)
    assert fits(tile, N, F, H, W, H, W, k, k - 1 - p)
    ld, pitch = B.conv_dy_rows_layout(d)
    rows, _ = B.relu_backward_rows(torch.ones_like(dY), dY, ld=ld)
    packed = torch.empty(B.conv_packed_weights_bytes(d, B.PASS_BACKWARD_DATA), dtype=torch.uint8, device="cuda")
    B.conv_pack_weights([d], [B.PASS_BACKWARD_DATA], [Wt], [packed])
    dX = B.conv_backward_data_packed(d, dY, packed)
    assert torch.equal(B.conv_backward_data_rows(d, rows, packed), dX)
    image = N - 1
    one = oracle.conv_backward_data(oracle.shape(1, C, H, W, F, k, k, 1, p), host(dY)[image:], host(Wt))
    assert np.max(np.abs(host(dX)[image:] - one)) <= 2e-2 * np.max(np.abs(one))
    per = B.conv_backward_data_relu_rows_sums(d)
    assert per is not None and -(-N * H * W // 512) <= per <= -(-N * H * W // 128)   # not split, columns of the larger tiles
    got, sums = B.conv_backward_data_relu_rows(d, rows, packed, y_front)
    B.tuning_set(B.TUNE_FUSED_WHOLE, 1)
    expect, _ = B.relu_backward_rows(y_front, B.conv_backward_data_packed(d, dY, packed))
    assert torch.equal(got, expect)
    assert tuple(sums.shape) == (C, per)
    scale = np.abs(host(expect)).sum(axis=1) + 1e-30
    assert np.max(np.abs(host(sums).sum(axis=1) - host(expect).sum(axis=1)) / scale) <= 1e-5


# small batches on the larger tiles, where the library's own choice is a small one: split reductions with one and four
# results per thread of the summing launch, both pitches of their patch
@pytest.mark.parametrize("N,C,H,W,F,k,p", [(3, 64, 9, 9, 37, 3, 1), (9, 64, 15, 15, 200, 3, 1), (5, 288, 13, 13, 384, 3, 1), (5, 96, 27, 27, 64, 5, 2)])
def test_larger_tiles_on_small_batches(B, N, C, H, W, F, k, p):
    rng = np.random.default_rng(C + F)
    X, Wt = wl.to_bf16_values(rng.standard_normal((N, C, H, W))), wl.to_bf16_values(0.05 * rng.standard_normal((F, C, k, k)))
    b = (0.05 * rng.standard_normal(F)).astype(np.float32)
    d = B.conv_desc(N, C, H, W, F, k, k, 1, p, 1, B.FLAG_FUSED)
    ref = oracle.conv_forward(oracle.shape(N, C, H, W, F, k, k, 1, p), X, Wt, b)
    B.tuning_set(B.TUNE_FUSED_WHOLE, 1)
    try:
        Y = B.conv_forward(d, gpu(X), gpu(Wt), torch.from_numpy(b).cuda())
        B.tuning_set(B.TUNE_FUSED_PITCH, 1)
        bare = B.conv_forward(d, gpu(X), gpu(Wt), torch.from_numpy(b).cuda())
    finally:
        B.tuning_set(B.TUNE_FUSED_PITCH, 0)
        B.tuning_set(B.TUNE_FUSED_WHOLE, 0)
    assert torch.equal(Y, bare)
    assert np.all(np.abs(host(Y) - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-4 * np.max(np.abs(ref)))


def test_knob_values(B):
    assert B._lib.omni_tuning_set(B.TUNE_FUSED_WHOLE, 6) == -1 and B._lib.omni_tuning_set(B.TUNE_FUSED_WHOLE, -1) == -1
