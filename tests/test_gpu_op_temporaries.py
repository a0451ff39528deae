"""Layer calls whose temporaries share one allocation, are divided over several
(each below 2 MB, together not) or take a mapped one: an image padded to 8
channels beside its packed filter, and weight gradients beside their split
partials.  Reference: the same sums in float64 over the bfloat16 operands.  An
output sums n products in float32 (n 2^-24 sum |x w|); a bfloat16 one is
rounded once more (2^-8 of its value)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [64, 178, 256])
def test_image_convolution(H):
    import torch
    import torch.nn.functional as F
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(H)
    x = torch.randn(4, H, H, 3, generator=gen).bfloat16()
    w = torch.randn(64, 3, 7, 7, generator=gen).bfloat16().float()
    y = binding.ekya_op_conv2d(x.cuda(), w.cuda(), 2, 3).cpu().double()
    xd, wd = x.double().permute(0, 3, 1, 2), w.double()
    ref = F.conv2d(xd, wd, stride=2, padding=3).permute(0, 2, 3, 1)
    bound = 147 * 2.0 ** -24 * F.conv2d(xd.abs(), wd.abs(), stride=2, padding=3).permute(0, 2, 3, 1)
    assert ((y - ref).abs() <= bound + 2.0 ** -8 * (ref.abs() + bound)).all()


@pytest.mark.parametrize("N,C,K", [(2, 64, 128), (40, 64, 128), (40, 256, 512)])
def test_weight_gradient(N, C, K):
    import torch
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(N + C)
    x, dy = torch.randn(N, 36, 36, C, generator=gen).bfloat16(), torch.randn(N, 36, 36, K, generator=gen).bfloat16()
    dw = binding.ekya_op_conv2d_wgrad(x.cuda(), dy.cuda(), (K, C, 1, 1), 1, 0).cpu().double().view(K, C)
    xd, dyd = x.double().view(-1, C), dy.double().view(-1, K)
    bound = N * 36 * 36 * 2.0 ** -24 * (dyd.abs().T @ xd.abs())
    assert ((dw - dyd.T @ xd).abs() <= bound).all()
