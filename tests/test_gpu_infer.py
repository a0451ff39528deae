"""Batched inference (sections 1 and 3.1, inference configurations) through
ekya_infer at the workload's resolutions against stored oracle logits: 520
drifting 224 px frames (two equal 260-frame chunks, so the chunk split runs),
resized to 224 (the stem reads the frames directly), 160 and 112 (resize
kernel, then the stem on the resized frames).  Labels equal the oracle's except where
its top-2 logit margin is below 2 tol x the frame's logit scale
max_j sum_i |W_ji f_i| (f the pooled features): a relative error tol in the
features -- 2e-2 for bf16 activations, 1e-5 for fp32 -- moves each logit by
at most tol times that scale, so two logits closer than twice it may swap.
(The stored classifiers remove the features' common direction, so the logits
are small residues of the features and their own relative error is several
times tol.)  The stored logits, scales and each case's classifier come from
tests/golden/make_infer_golden.py (oracle only)."""
import json
import os

import numpy as np
import pytest

from synth import WindowSpec, kaiming_resnet18_weights, make_frames
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "infer_224.json")
TOL = {"bf16": 2e-2, "f32": 1e-5}


@pytest.fixture(scope="module")
def golden():
    with open(GOLDEN) as f:
        return json.load(f)


@pytest.fixture(scope="module")
def ctx():
    from paper_2012_10557_amd import binding
    c = binding.ekya_create(0, 6)
    yield c
    binding.ekya_destroy(c)


def _weights(g, case):
    """The fixed-seed network with the case's stored classifier."""
    w = kaiming_resnet18_weights(seed=g["case"]["weights_seed"]).copy()
    fw = np.asarray(g["fc"][case]["weight"], dtype=np.float32).reshape(-1)
    fb = np.asarray(g["fc"][case]["bias"], dtype=np.float32)
    w[len(w) - fw.size - fb.size:len(w) - fb.size] = fw
    w[len(w) - fb.size:] = fb
    return w


@pytest.mark.parametrize("prec,res", [("bf16", 224), ("bf16", 160), ("bf16", 112), ("f32", 224)])
def test_infer_labels_match_oracle(ctx, golden, prec, res):
    import torch
    from paper_2012_10557_amd import binding
    c = golden["case"]
    spec = WindowSpec(c["n_frames"], 0, c["px"], c["px"], drift=c["drift"], seed=c["window_seed"])
    frames, _ = make_frames(spec, c["n_frames"], 1, 2)
    logits = np.asarray(golden["logits"][f"{prec}_{res}"])
    ref = np.argmax(logits, axis=1)
    labels = binding.ekya_infer(ctx, torch.tensor(_weights(golden, f"{prec}_{res}"), device="cuda"),
                                to_dev(frames, prec), res)
    torch.cuda.synchronize()
    got = labels.cpu().numpy()
    srt = np.sort(logits, axis=1)
    margin = srt[:, -1] - srt[:, -2]
    tie = margin < 2 * TOL[prec] * np.asarray(golden["scale"][f"{prec}_{res}"])
    counts = np.bincount(ref, minlength=6)
    print(f"{prec} {res}px: {int((got == ref).sum())}/{len(ref)} labels equal, {int(tie.sum())} "
          f"within the tie margin, oracle class counts {counts.tolist()}")
    assert (counts > 0).sum() >= 3, "the stored case must exercise several classes"
    assert np.all((got == ref) | tie), np.nonzero((got != ref) & ~tie)


@pytest.mark.parametrize("classes", [1, 8, 9, 16, 17])
def test_labels_at_the_edges_of_the_fused_head(classes):
    """Pooling and classifier are one launch for up to 8 classes.  float32: a
    logit is within 1e-5 of its scale max_j sum_i |W_ji f_i| + |b_j|."""
    import torch
    from oracle.resnet18 import ResNet18
    from paper_2012_10557_amd import binding
    net = ResNet18(classes)
    w = kaiming_resnet18_weights(seed=5, n_classes=classes)
    frames, _ = make_frames(WindowSpec(21, 0, 40, 40, drift="drift", seed=4), 21, 1, 2)
    P = net.unpack(w)
    f = net.forward(P, frames.astype(np.float64), 0, 4, train=False, tape={})
    w[-classes:] = -P["fc.weight"] @ f.mean(0)  # labels of several classes
    P = net.unpack(w)
    logits = f @ P["fc.weight"].T + P["fc.bias"]
    scale = (np.abs(f) @ np.abs(P["fc.weight"]).T + np.abs(P["fc.bias"])).max(1)
    c = binding.ekya_create(0, classes)
    try:
        got = binding.ekya_infer(c, torch.tensor(w, device="cuda"), to_dev(frames, "f32"), 40).cpu().numpy()
    finally:
        binding.ekya_destroy(c)
    best = logits.max(1)
    assert len(np.unique(got)) > (classes > 1)
    assert np.all(best - logits[np.arange(21), got] <= 2 * TOL["f32"] * scale)
