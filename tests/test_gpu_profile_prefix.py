"""Frozen-prefix caches of several depths in one profiling call: a deeper
depth's cache continues from a shallower one's where both hold the same rows.
Every candidate's losses and accuracies must be bit for bit those of a call
with that candidate alone, whose cache is built from the frames."""
import pytest

from synth import WindowSpec, kaiming_resnet18_weights, make_window
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("depths", [[(3, 0.5), (2, 0.5), (1, 0.5)], [(1, 0.5), (5, 0.5)], [(2, 0.25), (1, 0.5), (4, 0.5)],
                                    [(6, 0.5), (1, 0.25), (2, 0.25), (2, 0.5)]])
def test_joint_caches_equal_separate_ones(depths, prec):
    import torch
    from paper_2012_10557_amd import binding
    win = make_window(WindowSpec(48, 20, 65, 65, drift="none", seed=2))
    fr, hf = to_dev(win["frames"], prec), to_dev(win["heldout_frames"], prec)
    lab, hl = (torch.tensor(win[k], device="cuda") for k in ("labels", "heldout_labels"))
    w = torch.tensor(kaiming_resnet18_weights(seed=0), device="cuda")
    cfgs = [{"k": k, "subsample_frac": f, "epochs": 1, "lr": 0.05, "batch": 8, "seed": 10 + i}
            for i, (k, f) in enumerate(depths)]
    ctx = binding.ekya_create(0, 6)
    try:
        # rows of a depth's cache follow its largest fraction: keep it in the single calls
        def largest(k):
            return max((c for c in cfgs if c["k"] == k), key=lambda c: c["subsample_frac"])
        joint = binding.ekya_profile(ctx, w, cfgs, fr, lab, hf, hl, 7, concurrent=False)
        for c, r in zip(cfgs, joint):
            alone = binding.ekya_profile(ctx, w, [c, largest(c["k"])], fr, lab, hf, hl, 7, concurrent=False)[0]
            assert r["epoch_loss"] == alone["epoch_loss"] and r["heldout_acc"] == alone["heldout_acc"]
    finally:
        binding.ekya_destroy(ctx)
