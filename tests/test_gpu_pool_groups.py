"""The 3 x 3 / stride 2 max-pool backward takes more planes per workgroup the more there are: no plane's gradient depends on how
many planes the call has, bit for bit, and the last planes (a short group) agree with torch's own pool in fp32."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1606_04487_amd import binding
    assert torch.cuda.is_available()
    return binding


# planes from one group to many, whose sizes follow from an estimate (five planes of 13 x 13 alone: one group, 511: groups of three,
# 5003 of ten), up to the largest groups, short last groups; 9 x 9: the smallest planes with 16 pooled values, 8 x 8: four tasks a
# plane, 7 x 7: nine values, which the rule leaves alone
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("planes,H,W", [(1, 13, 13), (5, 13, 13), (511, 13, 13), (976, 8, 8), (8308, 29, 30), (1025, 13, 13), (5003, 13, 13), (33001, 9, 9), (1540, 55, 55), (700, 27, 30), (3001, 7, 7)])
def test_planes_per_group(B, planes, H, W, dtype):
    g = torch.Generator().manual_seed(planes + W)
    x = torch.randn(planes, H, W, generator=g).to(dtype).cuda()
    y, argmax = B.maxpool_forward(x)
    dy = torch.randint(-8, 9, tuple(y.shape), generator=g).to(dtype).cuda()     # small whole numbers: every sum is exact
    dx = B.maxpool_relu_backward(dy, argmax, y, H, W)
    for i in (0, planes // 2, planes - 1):
        j = min(planes, i + 3)
        part = B.maxpool_relu_backward(dy[i:j].clone(), argmax[i:j].clone(), y[i:j].clone(), H, W)
        assert torch.equal(dx[i:j], part)
    xr = x[-3:].float().cpu().requires_grad_()                                   # few ties matter: both take the first maximum
    torch.nn.functional.max_pool2d(xr[None], 3, 2, ceil_mode=True)[0].backward(torch.where(y > 0, dy, torch.zeros_like(dy))[-3:].float().cpu())
    assert torch.equal(dx[-3:].float().cpu(), xr.grad)
