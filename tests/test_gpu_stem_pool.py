"""The fused eval-mode stem (convolution, BatchNorm, ReLU, max pool) at the
widths where it changes: each number of 16-column tiles, odd and even output
widths (the last window lacks its right column), odd frame widths (2-byte
loads), pool rows that do not fill a block, and channels whose BatchNorm scale
is negative.  Classifier-only retraining on the frozen prefix exposes the
features: the classifier's first update is lr * dz^T f.  bfloat16 activations
move f by at most 2e-2 RMS (the gate of the output layer's update elsewhere), too wide to notice one wrong border
column: the exact test below counts every pooled pixel."""
import numpy as np
import pytest

from oracle import ekya as oracle
from oracle.resnet18 import ResNet18
from synth import WindowSpec, kaiming_resnet18_weights, make_window
from tests.gpu_util import rounded, to_dev

pytestmark = pytest.mark.gpu

SIZES = [(32, 32), (33, 33), (36, 50), (57, 64), (64, 66), (40, 98), (47, 130), (34, 163), (60, 224), (33, 221)]


@pytest.mark.parametrize("H,W", SIZES)
def test_first_classifier_update_matches_oracle(H, W):
    import torch
    from paper_2012_10557_amd import binding
    net = ResNet18(6)
    w0 = kaiming_resnet18_weights(seed=1)
    named = net.unpack(w0)
    rs = np.random.default_rng(H * 300 + W)
    named["bn1.weight"][:] = rs.uniform(0.5, 1.5, 64) * rs.choice([-1.0, 1.0], 64)
    named["bn1.bias"][:] = rs.normal(0, 0.3, 64)
    w0 = np.concatenate([np.asarray(named[n], dtype=np.float32).reshape(-1) for n, _ in net.spec])
    win = make_window(WindowSpec(10, 2, H, W, drift="none", seed=3))
    fr, hf = to_dev(win["frames"], "bf16"), to_dev(win["heldout_frames"], "bf16")
    lab, hl = (torch.tensor(win[k], device="cuda") for k in ("labels", "heldout_labels"))
    ctx = binding.ekya_create(0, 6)
    try:
        w = torch.tensor(w0, device="cuda")
        binding.ekya_retrain(ctx, w, 1, fr, lab, hf, hl, 1.0, 1, 0.1, 0.0, 10, 0)
    finally:
        binding.ekya_destroy(ctx)
    ref = oracle.retrain(w0, 1, rounded(win["frames"], "bf16"), win["labels"],
                         rounded(win["heldout_frames"], "bf16"), win["heldout_labels"], 1.0, 1, 0.1, 0.0, 10, 0)
    a, b, z = (net.unpack(np.asarray(v, dtype=np.float64))["fc.weight"] for v in (w.cpu().numpy(), ref.weights, w0))
    err = np.linalg.norm(a - b) / np.linalg.norm(b - z)
    print(f"{H} x {W}: {err:.2e}")
    assert err <= 2e-2


@pytest.mark.parametrize("px", [32, 64, 144, 224])
def test_zero_scale_channels_skip_infinite_sums(px):
    """A BatchNorm scale of 0 makes a finite sum the shift and an infinite one
    NaN, which the pool's maximum skips: with every scale 0 and one infinite
    pixel in the last corner (each window that sees it holds finite sums too)
    the frames are classified as they are without it, here by the classifier's
    bias.  A pooled -inf would make every logit NaN."""
    import torch
    from paper_2012_10557_amd import binding
    net = ResNet18(6)
    named = net.unpack(kaiming_resnet18_weights(seed=1))
    named["bn1.weight"][:] = 0.0
    named["bn1.bias"][:] = np.random.default_rng(px).uniform(0.1, 1.0, 64)
    named["fc.weight"][:] *= 1e-3
    named["fc.bias"][:] = [0, 0, 0, 0, 1, 0]
    w = torch.tensor(net.pack(named), dtype=torch.float32, device="cuda")
    frames = torch.randn(3, px, px, 3, generator=torch.Generator().manual_seed(px)).to(torch.bfloat16)
    frames[0, -1, -1, 0] = float("inf")
    frames[1, -1, -1, 1] = float("-inf")
    ctx = binding.ekya_create(0, 6)
    try:
        labels = binding.ekya_infer(ctx, w, frames.cuda(), px)
    finally:
        binding.ekya_destroy(ctx)
    assert labels.tolist() == [4, 4, 4]


def counting_network(rs, classes, zero_scale):
    """A network whose frozen stages add up the stem's pooled pixels: filters of
    -1, 0 and 1 in the stem, which BatchNorm multiplies by 1 or -1 (or 0) and
    shifts by a whole number, blocks that pass their input on, and 2 x 2 sums of
    the first 64 channels where a stage halves its size."""
    net = ResNet18(classes)
    named = net.unpack(kaiming_resnet18_weights(seed=1, n_classes=classes))
    for n, v in named.items():
        last = n.rsplit(".", 1)[1]
        if v.ndim == 4 or n.startswith("fc.") or last in ("bias", "running_mean"):
            v[:] = 0.0
        elif last == "running_var":
            v[:] = 1.0
        else:
            v[:] = np.sqrt(1.0 + 1e-5)  # folded scale 1 up to rounding
    named["conv1.weight"][:] = rs.choice([-1.0, 0.0, 1.0], (64, 3, 7, 7), p=[0.15, 0.7, 0.15])
    sign, shift = rs.choice([-1.0, 1.0], 64), rs.integers(-1, 2, 64).astype(np.float64)
    if zero_scale:
        sign[40], shift[40] = 0.0, 1.0
    named["bn1.weight"][:] *= sign
    named["bn1.bias"][:] = shift
    one = np.eye(64)
    for l in (2, 3, 4):
        named[f"layer{l}.0.conv1.weight"][:64, :64, 1:, 1:] = one[:, :, None, None]
        named[f"layer{l}.0.conv2.weight"][:64, :64, 1, 1] = one
    return net, named, sign, shift


#        N, H, W, a channel of scale 0 (its wave applies scale and shift to every sum)
COUNTED = [(300, 33, 33, False), (3, 34, 64, True), (150, 58, 90, False), (130, 63, 128, True), (135, 60, 147, False),
           (70, 120, 160, False), (135, 60, 193, True), (66, 113, 224, False), (5, 40, 221, False)]


@pytest.mark.parametrize("N,H,W,zero_scale", COUNTED)
def test_every_pooled_pixel_is_exact(N, H, W, zero_scale):
    """Whole numbers small enough for bfloat16 all the way, so the sum of the
    pooled pixels is exact for every frame and channel: at each number of
    column tiles, odd and even output widths, both kinds of input loads, and
    both with a block to each item and with more items than blocks (a block's
    LDS rows follow the previous item's).  A frame's features are read from the
    first update of a classifier of zeros in which each frame is a class of its
    own."""
    import torch
    import torch.nn.functional as F
    from paper_2012_10557_amd import binding
    rs = np.random.default_rng(N + W)
    classes = N + 1
    net, named, sign, shift = counting_network(rs, classes, zero_scale)
    x = (rs.random((N, H, W, 3)) < 0.02).astype(np.float32)
    t = torch.tensor(x).permute(0, 3, 1, 2)
    y = F.conv2d(t, torch.tensor(named["conv1.weight"]).float(), stride=2, padding=3)
    y = (y * torch.tensor(sign).float()[None, :, None, None] + torch.tensor(shift).float()[None, :, None, None]).relu()
    y = F.max_pool2d(y, 3, 2, 1)
    for _ in range(3):
        y = F.pad(y, (0, y.shape[3] % 2, 0, y.shape[2] % 2))
        y = y[:, :, ::2, ::2] + y[:, :, 1::2, ::2] + y[:, :, ::2, 1::2] + y[:, :, 1::2, 1::2]
    assert y.max() <= 256  # every whole number up to 256 is a bfloat16
    want = y.sum((2, 3)).numpy()
    w = torch.tensor(net.pack(named), dtype=torch.float32, device="cuda")
    fr, hf = torch.tensor(x, dtype=torch.bfloat16, device="cuda"), torch.zeros(1, H, W, 3, dtype=torch.bfloat16, device="cuda")
    lab, hl = torch.arange(N, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    ctx = binding.ekya_create(0, classes)
    try:
        binding.ekya_retrain(ctx, w, 1, fr, lab, hf, hl, 1.0, 1, float(N), 0.0, N, 0)
    finally:
        binding.ekya_destroy(ctx)
    fc = net.unpack(w.cpu().numpy().astype(np.float64))["fc.weight"]
    # class n gained f_n - mean softmax-weighted f, the last class only the latter
    got = (fc[:N, :64] - fc[N, :64]) * (y.shape[2] * y.shape[3])
    assert np.abs(got - np.round(got)).max() < 0.25
    np.testing.assert_array_equal(np.round(got), want)
