"""Trainable constant-Q plans: the kernel for batches of few workgroups adds the same terms in the same order as the one for large
batches, so a waveform's rows are the same bit for bit in either (kernels of one tap block to many hops, hops below and above a
chunk, ends that fall inside a run of four samples)."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sr,hop,fmin,n_bins,bpo,L", [(8000, 64, 60.0, 40, 12, 9001), (8000, 8, 200.0, 9, 12, 2050),
                                                      (8000, 48, 100.0, 30, 24, 7003), (22050, 512, 65.4, 60, 12, 40000)])
@pytest.mark.parametrize("fmt", ["MAGNITUDE", "COMPLEX"])
def test_few_frames_match_many(sr, hop, fmin, n_bins, bpo, L, fmt):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] cqt few {sr} {hop} {n_bins} {fmt}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_trainable(nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo,
                                                 fmt=getattr(nb, "NNA_OUT_" + fmt), device=0))
    x = torch.randn((1, L), generator=torch.Generator().manual_seed(hop)).cuda()
    few = nb.nna_cqt(plan, x)
    many = nb.nna_cqt(plan, x.repeat(256 * 256 // few.shape[2] + 1, 1))  # 256 tiles of 256 frames and more
    assert torch.isfinite(few).all()
    assert torch.equal(many[0], few[0]) and torch.equal(many[-1], few[0])


@pytest.mark.parametrize("sr,hop,n_bins,bpo,B", [(16000, 128, 24, 24, (81, 86)), (22050, 256, 252, 36, (36, 39)), (22050, 512, 84, 12, (430, 440))])
def test_line_between_the_kernels(sr, hop, n_bins, bpo, B):
    """Batches either side of 50,000 frames times the longest workgroup's share of the steps, the line of the kernel whose samples go
    through LDS: where it does not run (kernels of 132 and 136 hops) the smaller batch used to take 1.9 and 1.3 times as long as the larger."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] cqt few line {sr} {hop} {n_bins}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_trainable(nb.nna_plan_cqt(sr=sr, hop=hop, fmin=32.7, n_bins=n_bins, bins_per_octave=bpo, device=0))
    best = []
    for b in B:
        x = torch.randn((b, max(2 * sr, 3 * plan.info()["taps"] // 4)), generator=torch.Generator().manual_seed(b)).cuda()
        times = []
        for _ in range(8):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            nb.nna_cqt(plan, x)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        best.append(min(times))
    assert best[0] < 1.15 * best[1]
