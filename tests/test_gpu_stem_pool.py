"""The fused eval-mode stem (convolution, BatchNorm, ReLU, max pool) at the
widths where it changes: each number of 16-column tiles, odd and even output
widths (the last window lacks its right column), odd frame widths (2-byte
loads), pool rows that do not fill a block, and channels whose BatchNorm scale
is negative.  Classifier-only retraining on the frozen prefix exposes the
features: the classifier's first update is lr * dz^T f.  bfloat16 activations
move f by at most 2e-2 RMS (the gate of the output layer's update elsewhere)."""
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
