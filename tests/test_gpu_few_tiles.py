"""Trainable constant-Q plans on a grid of hops: batches of few workgroups, through 32 columns of the hops in LDS, against the kernel for
large batches bit for bit: tiles across waveforms, ends that fall inside a run of four samples, one kernel, no padding, more rows of a
hop than the LDS takes."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sr,hop,fmin,n_bins,bpo,B,L,center", [
    (8000, 64, 60.0, 40, 12, 5, 2306, True), (8000, 64, 60.0, 40, 12, 3, 2051, True), (8000, 32, 300.0, 1, 12, 70, 513, True),
    (16000, 96, 80.0, 30, 12, 2, 9000, False), (22050, 512, 65.4, 50, 12, 1, 20482, True), (8000, 32, 40.0, 17, 24, 9, 5003, True)])
def test_few_frames_match_many(sr, hop, fmin, n_bins, bpo, B, L, center):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] cqt few tiles {sr} {hop} {n_bins} {B}x{L}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, center=center, fmt=nb.NNA_OUT_COMPLEX, device=0)
    L = max(L, plan.info()["taps"] // (2 if center else 1) + 3)
    plan = nb.nna_plan_trainable(plan)
    x = torch.randn((B, L), generator=torch.Generator().manual_seed(hop + L)).cuda()
    few = nb.nna_cqt(plan, x)
    n = 256 * 256 // few.shape[2] // B + 1  # 256 tiles of 256 frames and more
    many = nb.nna_cqt(plan, x.repeat(n, 1))
    assert torch.isfinite(few).all()
    assert torch.equal(many[:B], few) and torch.equal(many[-B:], few)
