"""Fully connected layers at the sizes where the tiled kernel changes: tile
edges and remainders (16 and 32 wide), reductions shorter than one MFMA step,
not a multiple of 16 or of the chunks in flight, operands not 16-byte aligned,
both tile sizes, reductions of up to 64 elements in both (one chunk in flight),
and the edges of the block per row that few outputs without 16-byte loads take.
Reference: the same products in float64.  An output is sum_k a_k b_k in float32 in
some order, so it may be off by K 2^-24 sum |a b|."""
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (3, 5, 2), (16, 16, 16), (17, 33, 15), (64, 512, 6), (37, 501, 77), (31, 512, 129),
         (128, 516, 500), (400, 1024, 6), (513, 512, 1000), (5, 4096, 6), (1100, 40, 300),
         (33, 512, 520), (64, 520, 600), (65, 520, 600),
         (1024, 77, 8), (1025, 77, 8), (1025, 2049, 3), (40, 301, 9), (300, 512, 1),
         (90, 1025, 16), (1025, 1025, 9)]


def _close(got, ref, a, b, K):
    bound = K * 2.0 ** -24 * (a.double().abs() @ b.double().abs()) + 1e-30
    assert ((got.double() - ref).abs() <= bound).all()


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("N,I,J", SIZES)
def test_linear_matches_float64(N, I, J, offset):
    import torch
    from paper_2012_10557_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(N * 7 + I + J)

    def rand(*shape):  # offset 1: data 4 bytes past a 16-byte boundary
        n = torch.Size(shape).numel()
        return torch.randn(n + offset, generator=gen, device="cuda")[offset:].view(*shape)
    f, W, b, dz = rand(N, I), rand(J, I), rand(J), rand(N, J)
    z = binding.ekya_op_linear(f, W, b)
    ref = f.double() @ W.double().t() + b.double()
    ones = torch.ones(N, 1, device="cuda")
    _close(z, ref, torch.cat([f, ones], 1), torch.cat([W, b[:, None]], 1).t(), I + 1)
    df, dW, db = binding.ekya_op_linear_backward(dz, f, W)
    _close(df, dz.double() @ W.double(), dz, W, J)
    _close(dW, dz.double().t() @ f.double(), dz.t(), f, N)
    _close(db[:, None], dz.double().sum(0)[:, None], dz.t(), ones, N)


@pytest.mark.parametrize("N", [(1 << 24) - 1, 1 << 24])
def test_one_output_of_more_rows_than_a_launch_has_blocks(N):
    import torch
    from paper_2012_10557_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(1)
    f, W, b = (torch.randn(*s, generator=gen, device="cuda") for s in ((N, 3), (1, 3), (1,)))
    z = binding.ekya_op_linear(f, W, b)
    ref = f.double() @ W.double().t() + b.double()
    mag = f.double().abs() @ W.double().abs().t() + b.double().abs()
    assert ((z.double() - ref).abs() <= 4 * 2.0 ** -24 * mag).all()
