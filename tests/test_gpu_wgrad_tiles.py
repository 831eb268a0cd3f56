"""The tiles of the 13 x 13 layers' model gradient (shares of the reduction added through LDS) against the oracle."""
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


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


# one to three images in one range (a pair, its first half alone, a pair and a half) and several ranges of uneven length; one
# and several tiles of filters and channels; the bias gradient in the product's launch and in the sums'
@pytest.mark.parametrize("tile", [1, 2])
@pytest.mark.parametrize("N,C,F,splits", [(1, 64, 128, 0), (2, 128, 128, 1), (3, 64, 256, 1), (5, 64, 128, 2), (9, 128, 256, 0), (4, 64, 128, 4)])
def test_model_gradient_tiles(B, tile, N, C, F, splits):
    print("wgrad tile", tile, N, C, F, splits, flush=True)
    rng = np.random.default_rng(N + F)
    X, dY = wl.to_bf16_values(rng.standard_normal((N, C, 13, 13))), wl.to_bf16_values(rng.standard_normal((N, F, 13, 13)))
    s = oracle.shape(N, C, 13, 13, F, 3, 3, 1, 1)
    d = B.conv_desc(N, C, 13, 13, F, 3, 3, 1, 1, 1, B.FLAG_FUSED)
    ref, ref_b = oracle.conv_backward_weights(s, X, dY), oracle.bias_grad(s, dY)
    B.tuning_set(B.TUNE_WGRAD_TILE, tile)
    B.tuning_set(B.TUNE_WGRAD_SPLITS, splits)
    try:
        dW = torch.full((F, C, 3, 3), float("nan"), device="cuda")
        db = torch.full((F,), float("nan"), device="cuda")
        B.conv_backward_weights(d, gpu(X), gpu(dY), dW, db)
        again, none = B.conv_backward_weights(d, gpu(X), gpu(dY), want_dbias=False)
    finally:
        B.tuning_set(B.TUNE_WGRAD_TILE, 0)
        B.tuning_set(B.TUNE_WGRAD_SPLITS, 0)
    # fp32 sums of at most N x 169 products: a few 1e-7 of the gradient's scale
    assert np.max(np.abs(host(dW) - ref)) <= 1e-5 * np.max(np.abs(ref))
    assert np.max(np.abs(host(db) - ref_b)) <= 1e-5 * np.max(np.abs(ref_b))
    assert none is None and torch.equal(again, dW)


# the tile without shares, which the library takes itself where the others' tiles fill the chip badly: one range of one image and
# of a pair and a half against the oracle, three and five ranges of uneven length against a forced tile
@pytest.mark.parametrize("N,C,F", [(1, 832, 1280), (3, 832, 1280), (18, 832, 640), (29, 256, 1408)])
def test_tile_without_shares(B, N, C, F):
    print("wgrad whole tile", N, C, F, flush=True)
    rng = np.random.default_rng(N + F)
    X, dY = gpu(wl.to_bf16_values(rng.standard_normal((N, C, 13, 13)))), gpu(wl.to_bf16_values(rng.standard_normal((N, F, 13, 13))))
    d = B.conv_desc(N, C, 13, 13, F, 3, 3, 1, 1, 1, B.FLAG_FUSED)
    dW, db = B.conv_backward_weights(d, X, dY)
    B.tuning_set(B.TUNE_WGRAD_TILE, 1)
    try:
        ref, ref_b = (host(t) for t in B.conv_backward_weights(d, X, dY))
    finally:
        B.tuning_set(B.TUNE_WGRAD_TILE, 0)
    if N <= 3:
        s = oracle.shape(N, C, 13, 13, F, 3, 3, 1, 1)
        ref, ref_b = oracle.conv_backward_weights(s, host(X), host(dY)), oracle.bias_grad(s, host(dY))
    assert np.max(np.abs(host(dW) - ref)) <= 1e-5 * np.max(np.abs(ref))
    assert np.max(np.abs(host(db) - ref_b)) <= 1e-5 * np.max(np.abs(ref_b))


def test_knob_values(B):
    assert B._lib.omni_tuning_set(B.TUNE_WGRAD_TILE, 3) == -1 and B._lib.omni_tuning_set(B.TUNE_WGRAD_TILE, -1) == -1
