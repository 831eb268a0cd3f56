"""Launch shapes at their edges, against the oracle: work split finely because a layer is small, tiles that a layer
fills only partly, remainders on both sides of a tile."""
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
