"""Max-pool of whole channel vectors: windows of one and of several batches of taps, odd sizes, images of one row, and values at the
type's ends (the lowest number, infinities): bit for bit the winning input."""
import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("win,stride,pad,H,W,C", [(1, 1, 0, 3, 5, 8), (2, 2, 0, 7, 6, 16), (2, 1, 1, 4, 4, 8), (3, 2, 1, 15, 14, 72), (4, 3, 2, 9, 1, 8), (5, 1, 2, 6, 7, 24), (7, 4, 3, 33, 31, 8)])
def test_windows(win, stride, pad, H, W, C, dtype):
    import torch
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    gen = torch.Generator().manual_seed(win * 10 + stride)
    x = (torch.rand((3, H, W, C), generator=gen) * 2 - 1).to(dt)
    x[1] = float("-inf")
    x[2] = torch.finfo(dt).min
    x[2, H // 2, W // 2, ::3] = float("inf")
    ref = torch.nn.functional.max_pool2d(x.double().permute(0, 3, 1, 2), win, stride, min(pad, win // 2)).permute(0, 2, 3, 1)
    assert pad <= win // 2
    P, Q = ref.shape[1:3]
    big = torch.full((ref.numel() + 16,), 7.0, dtype=dt, device="cuda")
    y = big[8:8 + ref.numel()].view(3, P, Q, C)
    dx = x.cuda()
    sc.st_maxpool_nhwc(dx, y, 3, H, W, C, win, stride, pad, dtype)
    torch.cuda.synchronize()
    assert torch.equal(y.cpu().double(), ref)
    assert (big[:8] == 7).all() and (big[-8:] == 7).all()
