"""Lowering and col2im of stride-1 layers whose output is as wide as the input, which run straight from memory: bit-exact
against the oracle's index map, resp. against its scatter."""
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


def gpu(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return t.to(torch.bfloat16) if dtype == 1 else t


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


# planes as narrow as the direct form takes (16 bytes of pixels and two) and one narrower, odd and even; pieces over the ends
# of rows, images and tensors; windows of 1, 3 and 5, taller and flatter than wide, heights that shrink; one column; fewer
# pieces of work than XCDs, and a number that eight ranges do not divide; 5 x 5 windows of one round of staged workgroups and
# of one more image, pixel or channel
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("N,C,H,W,kh,kw,ph,pw", [(3, 2, 5, 6, 3, 3, 1, 1), (3, 2, 5, 5, 3, 3, 1, 1), (5, 3, 3, 10, 5, 5, 2, 2), (2, 3, 7, 9, 5, 5, 2, 2),
                                                (4, 5, 13, 13, 3, 3, 1, 1), (1, 1, 2, 11, 3, 3, 1, 1), (7, 2, 9, 12, 1, 1, 0, 0), (2, 4, 9, 14, 5, 3, 0, 1),
                                                (3, 2, 6, 13, 1, 5, 0, 2), (1, 3, 27, 27, 5, 5, 2, 2), (2, 2, 4, 31, 3, 5, 2, 2), (9, 37, 19, 21, 3, 3, 1, 1),
                                                (70, 3, 11, 10, 5, 5, 2, 2), (1, 256, 16, 16, 5, 5, 2, 2),
                                                (1, 3, 17, 16, 5, 5, 2, 2), (1, 385, 7, 10, 5, 5, 2, 2), (2, 5, 12, 11, 5, 5, 2, 2)])
def test_lowering_and_col2im(B, N, C, H, W, kh, kw, ph, pw, dtype):
    rng = np.random.default_rng(N * W + kh)
    X = wl.to_bf16_values(rng.standard_normal((N, C, H, W)))
    s = oracle.shape(N, C, H, W, 4, kh, kw, (1, 1), (ph, pw))
    d = B.conv_desc(N, C, H, W, 4, kh, kw, (1, 1), (ph, pw), dtype)
    ref = oracle.lower(s, X)
    K, M = ref.shape
    for ld in (B.conv_dhat_ld(d), (M + 7) // 8 * 8):
        D = torch.full((K, ld), float("nan"), dtype=B.torch_dtype(dtype), device="cuda")
        B.lower(d, gpu(X, dtype), D, ld)
        assert np.array_equal(host(D)[:, :M], ref) and not host(D)[:, M:].any()
    G = wl.to_bf16_values(rng.standard_normal((K, M)))
    want = oracle.col2im(s, G)
    for ld in (M, M + 3, M + 8):       # the matrix ends with its last column; what lies behind the others is no number
        Gd = torch.full((K * ld - (ld - M) + 64,), float("nan"), dtype=B.torch_dtype(dtype), device="cuda")
        torch.as_strided(Gd, (K, M), (ld, 1)).copy_(gpu(G, dtype))
        dX = torch.full((N, C, H, W), float("nan"), dtype=B.torch_dtype(dtype), device="cuda")
        B.col2im(d, Gd, dX, ld)
        # fp32 sums of at most 25 terms, one rounding to bf16
        assert np.all(np.abs(host(dX) - want) <= (2.0 ** -8 if dtype == 1 else 0.0) * np.abs(want) + 1e-5)


# a lowered matrix beyond the caches is stored past them: 210 MB are not, 262 MB are
@pytest.mark.parametrize("dtype,N", [(0, 128), (1, 256), (0, 160), (1, 320)])
def test_lowering_past_the_caches(B, dtype, N):
    C, H = 64, 16
    rng = np.random.default_rng(N)
    X = wl.to_bf16_values(rng.standard_normal((N, C, H, H)))
    d = B.conv_desc(N, C, H, H, 4, 5, 5, 1, 2, dtype)
    D = B.lower(d, gpu(X, dtype), None, B.conv_dhat_ld(d))
    ref = oracle.lower(oracle.shape(N, C, H, H, 4, 5, 5, 1, 2), X)
    step = 100                         # rows compared at a time
    for k in range(0, ref.shape[0], step):
        assert np.array_equal(host(D[k:k + step]), ref[k:k + step])


# One column of windows per channel and 2^26 + 1 channels: more workgroups than a grid dimension can hold (2^32 threads).
# D-hat of a 1 x 1 window is X, row by row.
def test_more_channels_than_a_grid_dimension(B):
    if torch.cuda.mem_get_info()[0] < 12 * 2 ** 30:
        pytest.skip("needs 12 GB of free device memory")
    C, W, ld = 2 ** 26 + 1, 10, 16
    d = B.conv_desc(1, C, 1, W, 1, 1, 1, 1, 0, B.BF16)
    X = torch.randint(-99, 100, (1, C, 1, W), dtype=torch.int8, device="cuda").to(torch.bfloat16)
    D = B.lower(d, X, torch.full((C, ld), float("nan"), dtype=torch.bfloat16, device="cuda"), ld)
    assert torch.equal(D[:, :W], X.view(C, W)) and not bool(D[:, W:].any())
