"""Forward convolutions with few output pixels, at each tile the kernel picks
(16 x 32, 32 x 32, 32 x 64, 64 x 64) and at its edges: one output pixel, tile
remainders in channels and pixels, strides, wide filters, 1 x 1 filters, odd
sizes, and reductions that do not divide evenly over the waves.  Reference: the
convolution in float64 over the same (bfloat16-rounded) operands.  An output
sums n products in float32, so it may be off by n 2^-24 sum |x w|, and in
bfloat16 is rounded once more (2^-8 of its value)."""
import pytest

pytestmark = pytest.mark.gpu

#        N, H, W, C, K, R, stride
SHAPES = [(1, 1, 1, 64, 64, 3, 1), (1, 7, 7, 512, 512, 3, 1), (4, 14, 14, 256, 256, 3, 1),
          (4, 28, 28, 128, 128, 3, 1), (16, 28, 28, 128, 128, 3, 1), (3, 13, 9, 192, 72, 5, 2),
          (5, 6, 11, 512, 1000, 1, 1), (7, 15, 15, 128, 256, 3, 2), (2, 9, 40, 64, 136, 3, 1),
          (9, 20, 20, 64, 128, 3, 2)]


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("N,H,W,C,K,R,stride", SHAPES)
def test_few_pixel_convolution_matches_float64(N, H, W, C, K, R, stride, prec):
    import torch
    import torch.nn.functional as F
    from paper_2012_10557_amd import binding
    dtype = torch.float32 if prec == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(N + H + C + K)
    x = torch.randn(N, H, W, C, generator=gen).to(dtype)
    w = torch.randn(K, C, R, R, generator=gen).to(dtype).float()
    y = binding.ekya_op_conv2d(x.cuda(), w.cuda(), stride, R // 2).cpu().double()
    xd, wd = x.double().permute(0, 3, 1, 2), w.double()
    ref = F.conv2d(xd, wd, stride=stride, padding=R // 2).permute(0, 2, 3, 1)
    mag = F.conv2d(xd.abs(), wd.abs(), stride=stride, padding=R // 2).permute(0, 2, 3, 1)
    bound = C * R * R * 2.0 ** -24 * mag
    if prec == "bf16":
        bound = bound + 2.0 ** -8 * (ref.abs() + bound)
    assert ((y - ref).abs() <= bound + 1e-30).all()


def test_image_beyond_32_bit_offsets():
    """One float32 image of 2^31 elements, whose offsets need 64 bits."""
    import torch
    from paper_2012_10557_amd import binding
    H, C, K, stride = 2048, 512, 4, 64
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(1, H, H, C, generator=gen, device="cuda")
    w = torch.randn(K, C, 3, 3, generator=gen, device="cuda")
    y = binding.ekya_op_conv2d(x, w, stride, 1).double()
    at = torch.arange(0, H, stride, device="cuda")
    ref, mag = torch.zeros_like(y[0]), torch.zeros_like(y[0])
    for r in range(3):
        for s in range(3):
            h, v = (at - 1 + r)[:, None], (at - 1 + s)[None, :]
            px = x[0, h.clamp(min=0), v.clamp(min=0)].double() * ((h >= 0) & (v >= 0))[..., None]
            ref += px @ w[:, :, r, s].double().T
            mag += px.abs() @ w[:, :, r, s].double().abs().T
    assert ((y[0] - ref).abs() <= C * 9 * 2.0 ** -24 * mag).all()


# measured with split tiles, whose fp32 chains are shorter: relative error
# against float64 of the same shapes
@pytest.mark.parametrize("H,C,N,split", [(14, 256, 16, 2.50e-7), (2, 512, 48, 2.15e-7), (8, 128, 48, 1.55e-7)])
def test_f32_sums_round_no_worse_than_split_tiles(H, C, N, split):
    """A float32 output in one chain of n products has 1.3 to 1.7 times the
    rounding error of the split tiles; sums kept in runs have less."""
    import torch
    import torch.nn.functional as F
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(C)
    x, w = torch.randn(N, H, H, C, generator=gen).relu(), torch.randn(C, C, 3, 3, generator=gen)
    y = binding.ekya_op_conv2d(x.cuda(), w.cuda(), 1, 1).cpu().double()
    ref = F.conv2d(x.double().permute(0, 3, 1, 2), w.double(), padding=1).permute(0, 2, 3, 1)
    err = ((y - ref).norm() / ref.norm()).item()
    print(f"{err:.2e}")
    assert err <= split
