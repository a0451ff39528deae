"""float32 convolutions with more than 448 tiles of 64 x 64, forward and data
gradient: tile remainders in channels and pixels, stride 2 with odd and even
sizes, 1 x 1 and 5 x 5 filters, 32 and 96 reduced channels; and 1 x 1 filters
of too few channels for the few-pixel kernel beyond 128 tiles, up to 448, on
the register-staged tiles, as do 3 x 3 filters whose 128 x 128 tiles fill
rounds of two per CU.  Reference: the same sums in float64.  An output sums n products in float32, so it may be off
by n 2^-24 sum |x w|."""
import pytest

pytestmark = pytest.mark.gpu

#        N, H, W, C, K, R, stride
SHAPES = [(19, 40, 40, 64, 64, 3, 1), (5, 57, 55, 96, 160, 3, 2), (9, 41, 40, 32, 96, 5, 2),
          (13, 26, 30, 160, 224, 1, 1), (33, 29, 31, 64, 96, 1, 2), (60, 7, 9, 128, 512, 3, 1)]
# 1 x 1: 314, 288 and 130 tiles forward
SHORT = [(25, 20, 20, 64, 128, 1, 1), (36, 31, 32, 128, 128, 1, 2), (3, 52, 53, 32, 64, 1, 1)]
# 512 tiles of 128 x 128, and 983 of 1024 (the last one partly filled)
FULL = [(16, 64, 64, 64, 128, 3, 1), (31, 45, 45, 96, 256, 3, 1)]


@pytest.mark.parametrize("N,H,W,C,K,R,stride", SHAPES + SHORT + FULL)
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


# relative error against float64 of register-staged tiles whose reduction is
# split in two or three, measured at the same shapes: forward, data gradient
SPLIT = [(10, 56, 64, 2.10e-7, 3.05e-7), (20, 28, 128, 2.54e-7, 3.51e-7), (40, 14, 256, 3.51e-7, 4.90e-7),
         (75, 7, 512, 4.80e-7, 6.80e-7)]


@pytest.mark.parametrize("N,H,C,fwd,dgrad", SPLIT)
def test_f32_sums_round_no_worse_than_split_tiles(N, H, C, fwd, dgrad):
    """At 449 to 511 tiles a split reduction would fill the chip; one chain of
    n products instead has 1.4 to 1.7 times its rounding error."""
    import torch
    import torch.nn.functional as F
    from torch.nn.grad import conv2d_input
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(C)
    x, w = torch.randn(N, H, H, C, generator=gen).relu(), torch.randn(C, C, 3, 3, generator=gen)
    dy = torch.randn(N, H, H, C, generator=gen)
    y = binding.ekya_op_conv2d(x.cuda(), w.cuda(), 1, 1)[:8].cpu().double()
    dx = binding.ekya_op_conv2d_dgrad(dy.cuda(), w.cuda(), (N, H, H, C), 1, 1)[:8].cpu().double()
    xd, dyd = (v[:8].double().permute(0, 3, 1, 2) for v in (x, dy))
    ref = F.conv2d(xd, w.double(), padding=1).permute(0, 2, 3, 1)
    rdx = conv2d_input(xd.shape, w.double(), dyd, 1, 1).permute(0, 2, 3, 1)
    err = [((a - b).norm() / b.norm()).item() for a, b in ((y, ref), (dx, rdx))]
    print(" ".join(f"{e:.2e}" for e in err))
    assert err[0] <= fwd and err[1] <= dgrad


#        N, H, C, K, R: few output pixels, 490 tiles, 1274 tiles
@pytest.mark.parametrize("N,H,C,K,R", [(3, 14, 64, 64, 3), (20, 28, 128, 128, 3), (52, 28, 64, 128, 1)])
def test_tensors_aligned_to_4_bytes(N, H, C, K, R):
    """float32 layer calls take tensors that do not start on 16 bytes: their
    loads are not direct 16-byte copies to LDS."""
    import torch
    import torch.nn.functional as F
    from torch.nn.grad import conv2d_input
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(N + C)

    def shifted(t):
        v = torch.zeros(t.numel() + 4, device="cuda")[1:1 + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 == 4 and v.is_contiguous()
        return v
    x, w = torch.randn(N, H, H, C, generator=gen), torch.randn(K, C, R, R, generator=gen)
    dy = torch.randn(N, H, H, K, generator=gen)
    y = binding.ekya_op_conv2d(shifted(x), w.cuda(), 1, R // 2).cpu().double()
    dx = binding.ekya_op_conv2d_dgrad(shifted(dy), w.cuda(), (N, H, H, C), 1, R // 2).cpu().double()
    xd, wd, dyd = x.double().permute(0, 3, 1, 2), w.double(), dy.double().permute(0, 3, 1, 2)
    ref = F.conv2d(xd, wd, padding=R // 2).permute(0, 2, 3, 1)
    mag = F.conv2d(xd.abs(), wd.abs(), padding=R // 2).permute(0, 2, 3, 1)
    assert ((y - ref).abs() <= C * R * R * 2.0 ** -24 * mag).all()
    ref = conv2d_input(xd.shape, wd, dyd, 1, R // 2).permute(0, 2, 3, 1)
    mag = conv2d_input(xd.shape, wd.abs(), dyd.abs(), 1, R // 2).permute(0, 2, 3, 1)
    assert ((dx - ref).abs() <= K * R * R * 2.0 ** -24 * mag).all()
