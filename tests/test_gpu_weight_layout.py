"""Weight layouts between the caller's [K][C][R][S] array and the kernels'
copies, at the filters where the copying changes: one tap, an even number of
taps, a row longer than a staged part (C R S > 4608), more taps than the
transposing tile takes (128) and more than a staged row (4608), channel counts
off the tile, and padded input channels.  The convolution of a unit impulse
reads every weight back, so the comparison is with the weights themselves:
exact in float32, rounded once in bfloat16."""
import pytest

pytestmark = pytest.mark.gpu

FILTERS = [(8, 64, 1, 1), (40, 64, 2, 2), (64, 64, 3, 3), (600, 64, 3, 3), (16, 128, 7, 9), (8, 64, 12, 11),
           (8, 64, 70, 70)]


def _impulse(n, H, W, C, h, w, dtype):
    import torch
    x = torch.zeros(n, H, W, C, dtype=dtype, device="cuda")
    for i in range(n):
        x[i, h, w, i] = 1
    return x


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("C,K,R,S", FILTERS)
def test_convolution_reads_every_weight(C, K, R, S, prec):
    import torch
    from paper_2012_10557_amd import binding
    dtype = torch.float32 if prec == "f32" else torch.bfloat16
    w = torch.randn(K, C, R, S, generator=torch.Generator().manual_seed(C + K + R)).cuda()
    want = w.to(dtype).permute(1, 2, 3, 0)  # [C][R][S][K]
    # image c: an impulse of channel c at the far corner; output (p, q) is the
    # weight of the tap that reaches it
    y = binding.ekya_op_conv2d(_impulse(C, 2 * R - 1, 2 * S - 1, C, R - 1, S - 1, dtype), w, 1, 0)
    assert torch.equal(y.flip(1, 2), want)
    # gradient k: an impulse of output channel k spreads w[k] over the input
    if K % 64 == 0:
        dx = binding.ekya_op_conv2d_dgrad(_impulse(K, 1, 1, K, 0, 0, dtype), w, (K, R, S, C), 1, 0)
        assert torch.equal(dx, want.permute(3, 1, 2, 0))


@pytest.mark.parametrize("C,K,R,S", [(3, 64, 7, 7)] + FILTERS[:5])
def test_weight_gradient_is_returned_in_the_callers_layout(C, K, R, S):
    import torch
    from paper_2012_10557_amd import binding
    gen = torch.Generator().manual_seed(C + R)
    x = torch.randn(1, R, S, C, generator=gen).cuda()
    dw = binding.ekya_op_conv2d_wgrad(x, _impulse(1, 1, 1, K, 0, 0, torch.float32), (K, C, R, S), 1, 0)
    assert torch.equal(dw[0], x[0].permute(2, 0, 1)) and not dw[1:].any()


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,classes", [(0, 6), (37, 5)])
def test_model_round_trip(hidden, classes, prec):
    """A loaded model exports the array it was loaded from, bit for bit."""
    import torch
    from paper_2012_10557_amd import binding
    n = binding.ekya_weights_count(classes, hidden)
    w = torch.randn(n, generator=torch.Generator().manual_seed(n)).cuda().abs()
    m = binding.ekya_model_create(0, classes, binding.EKYA_FP32 if prec == "f32" else binding.EKYA_BF16, hidden)
    try:
        binding.ekya_model_load(m, w)
        out = torch.empty_like(w)
        binding.ekya_model_export(m, out)
        torch.cuda.synchronize()
        assert torch.equal(out, w)
    finally:
        binding.ekya_model_destroy(m)
