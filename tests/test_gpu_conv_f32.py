"""float32 convolutions with more than 448 tiles of 64 x 64, forward and data
gradient: tile remainders in channels and pixels, stride 2 with odd and even
sizes, 1 x 1 and 5 x 5 filters, 32 and 96 reduced channels.  Reference: the
same sums in float64.  An output sums n products in float32, so it may be off
by n 2^-24 sum |x w|."""
import pytest

pytestmark = pytest.mark.gpu

#        N, H, W, C, K, R, stride
SHAPES = [(19, 40, 40, 64, 64, 3, 1), (5, 57, 55, 96, 160, 3, 2), (9, 41, 40, 32, 96, 5, 2),
          (13, 26, 30, 160, 224, 1, 1), (33, 29, 31, 64, 96, 1, 2), (60, 7, 9, 128, 512, 3, 1)]


@pytest.mark.parametrize("N,H,W,C,K,R,stride", SHAPES)
def test_f32_convolution_matches_float64(N, H, W, C, K, R, stride):
    import torch
    import torch.nn.functional as F
    from torch.nn.grad import conv2d_input
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(N + H + C + K)
    x = torch.randn(N, H, W, C, generator=gen)
    w = torch.randn(K, C, R, R, generator=gen)
    xd, wd = x.double().permute(0, 3, 1, 2), w.double()
    y = binding.ekya_op_conv2d(x.cuda(), w.cuda(), stride, R // 2).cpu().double()
    ref = F.conv2d(xd, wd, stride=stride, padding=R // 2).permute(0, 2, 3, 1)
    mag = F.conv2d(xd.abs(), wd.abs(), stride=stride, padding=R // 2).permute(0, 2, 3, 1)
    assert ((y - ref).abs() <= C * R * R * 2.0 ** -24 * mag).all()

    dy = torch.randn(*ref.shape, generator=gen)
    dyd = dy.double().permute(0, 3, 1, 2)
    dx = binding.ekya_op_conv2d_dgrad(dy.cuda(), w.cuda(), (N, H, W, C), stride, R // 2)
    dx = dx.cpu().double()
    ref = conv2d_input(xd.shape, wd, dyd, stride, R // 2).permute(0, 2, 3, 1)
    mag = conv2d_input(xd.shape, wd.abs(), dyd.abs(), stride, R // 2).permute(0, 2, 3, 1)
    assert ((dx - ref).abs() <= K * R * R * 2.0 ** -24 * mag + 1e-30).all()
