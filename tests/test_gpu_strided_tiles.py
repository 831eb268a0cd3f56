"""Tiles of the wide-stride kernels.  The forward kernel has three (128, 256 and 512 positions per workgroup): the number of
images decides which one runs, and no image's result may depend on it, bit for bit; the oracle holds the last images of each
case.  The model gradient has two row tiles, each held to the oracle."""
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


# (images, C, H, W, F, kh, kw, sh) and the images per call that keep the reference on the smallest tile
CASES = [
    (140, 2, 30, 41, 5, 3, 5, 2, 128),        # 140 positions: 2 small tiles per image; 256 positions, one each
    (257, 2, 30, 41, 5, 3, 5, 2, 128),        # 512 positions: one workgroup takes a second tile
    (64, 3, 99, 99, 64, 7, 7, 4, 32),         # 576 positions: 5 small tiles, 3 of 256 with a short one
    (140, 3, 99, 99, 64, 7, 7, 4, 32),        # 280 tiles of 512, the second of an image short
    (13, 3, 227, 227, 96, 11, 11, 4, 8),      # 55 x 55 outputs: rows cut by the tiles' edges, 96 filters, 23 steps
    (300, 1, 12, 9, 3, 2, 1, 1, 256),         # one channel, window of one column
]


@pytest.mark.parametrize("cfg", CASES)
def test_tiles_agree(B, cfg):
    N, C, H, W, F, kh, kw, sh, part = cfg
    rng = np.random.default_rng(41)
    X = wl.to_bf16_values(rng.standard_normal((N, C, H, W))).astype(np.float32)
    Wt = wl.to_bf16_values(0.05 * rng.standard_normal((F, C, kh, kw))).astype(np.float32)
    b = (0.05 * rng.standard_normal(F)).astype(np.float32)
    Xg, Wg, bg = torch.from_numpy(X).cuda().bfloat16(), torch.from_numpy(Wt).cuda().bfloat16(), torch.from_numpy(b).cuda()
    flags = B.FLAG_FUSED | B.FLAG_RELU

    def run(i, j):
        d = B.conv_desc(j - i, C, H, W, F, kh, kw, (sh, 4), (0, 0), B.BF16, flags)
        assert B.conv_fused_supported(d, B.PASS_FORWARD)
        return B.conv_forward(d, Xg[i:j].contiguous(), Wg, bg)

    got = run(0, N)
    for i in range(0, N, part):
        j = min(N, i + part)
        assert torch.equal(got[i:j], run(i, j))
    s = oracle.shape(2, C, H, W, F, kh, kw, (sh, 4), (0, 0))
    ref = np.maximum(oracle.conv_forward(s, X[-2:], Wt, b), 0)
    err = np.max(np.abs(got[-2:].float().cpu().numpy() - ref)) / np.max(np.abs(ref))
    assert err <= 2 ** -8     # the fp32 sums (errors below 1e-5 of the largest) rounded to bf16 once


@pytest.mark.parametrize("N,C,H,F,k", [(3, 3, 227, 96, 11),    # 32 filters per workgroup: 36 ranges, three row tiles
                                       (8, 3, 227, 96, 11),    # 96 filters: 96 ranges would be 288 workgroups of 32
                                       (24, 3, 131, 96, 7),    # the same without three groups per window row
                                       (24, 3, 131, 33, 7)])   # a second row tile of one filter
def test_model_gradient_row_tiles(B, N, C, H, F, k):
    rng = np.random.default_rng(43)
    Ho = (H - k) // 4 + 1
    X = wl.to_bf16_values(rng.standard_normal((N, C, H, H))).astype(np.float32)
    dY = wl.to_bf16_values(rng.standard_normal((N, F, Ho, Ho))).astype(np.float32)
    s = oracle.shape(N, C, H, H, F, k, k, (4, 4), (0, 0))
    d = B.conv_desc(N, C, H, H, F, k, k, 4, 0, B.BF16, B.FLAG_FUSED)
    assert B.conv_fused_supported(d, B.PASS_BACKWARD_WEIGHTS)
    dW, db = B.conv_backward_weights(d, torch.from_numpy(X).cuda().bfloat16(), torch.from_numpy(dY).cuda().bfloat16())
    # exact products in fp32 sums of N Ho Ho terms in ranges: far below sqrt(terms) 2^-24 of the largest sum
    for got, ref in ((dW, oracle.conv_backward_weights(s, X, dY)), (db, oracle.bias_grad(s, dY))):
        assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
