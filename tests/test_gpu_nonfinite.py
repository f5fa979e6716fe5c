"""Samples that are not finite, in the constant-Q calls that take a kernel's hop-blocks as combinations of a few functions: bins and
frames whose own taps lie clear of such a sample hold what they hold without it, those that meet it are not finite."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("sr,hop,fmin,n_bins,bpo,B,L,at", [
    (22050, 512, 32.7, 84, 12, 3, 40001, 20077), (8000, 64, 40.0, 40, 24, 4, 9000, 4321), (16000, 128, 60.0, 33, 24, 2, 16391, 3),
    (22050, 512, 32.7, 84, 12, 200, 22050, 22049)])
def test_reach_of_one_sample(sr, hop, fmin, n_bins, bpo, B, L, at, bad):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] nonfinite sr={sr} hop={hop} {n_bins} {B}x{L} {bad}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, fmt=nb.NNA_OUT_COMPLEX, device=0)
    assert nb.nna_plan_applied_tiles(plan, B, L)[0][0] > 0
    x = (0.3 * np.random.default_rng([43, hop, n_bins]).standard_normal((B, L))).astype(np.float32)
    b = B // 2
    x[b, at] = 0.0
    clean = nb.nna_cqt(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    x[b, at] = bad
    got = nb.nna_cqt(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(np.delete(got, b, 0), np.delete(clean, b, 0))
    got, clean = got[b].reshape(n_bins, 2, -1), clean[b].reshape(n_bins, 2, -1)
    re, im = oracle.cqt_kernels(sr, fmin, n_bins, bpo)
    K = re.shape[1]
    own = [(np.flatnonzero(re[k] ** 2 + im[k] ** 2).min(), np.flatnonzero(re[k] ** 2 + im[k] ** 2).max() + 1) for k in range(n_bins)]
    places = {K // 2 + at, K // 2 - at, K // 2 + 2 * (L - 1) - at}  # in the padded waveform: as stored, mirrored at either end
    frames = hop * np.arange(got.shape[2])
    tol = 1e-5 * np.abs(clean).max()
    for k in range(n_bins):
        # the kernels of eight neighbouring bins share their steps of 16 taps
        lo, hi = own[8 * (k // 8)][0] // 16 * 16, (own[8 * (k // 8)][1] + 15) // 16 * 16
        clear = np.all([(p < frames + lo - 16) | (p >= frames + hi + 16) for p in places], 0)
        meets = np.any([(p >= frames + own[k][0] + 2) & (p < frames + own[k][1] - 2) for p in places], 0)
        assert np.abs(got[k][:, clear] - clean[k][:, clear]).max(initial=0.0) <= tol, k
        assert not np.isfinite(got[k][:, meets]).any(), k


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 3.4e38])
@pytest.mark.parametrize("sr,hop,fmin,n_bins,bpo,B,L,at", [
    (22050, 512, 32.7, 84, 12, 2, 40001, 20077), (16000, 96, 50.0, 60, 12, 3, 9001, 4500), (22050, 512, 32.7, 84, 12, 200, 22050, 11270),
    (16000, 96, 50.0, 60, 12, 400, 9001, 4503)])
def test_short_kernels(sr, hop, fmin, n_bins, bpo, B, L, at, bad):
    """Bins taken tap by tap beside the others, for one and two frame blocks a wave: a sample reaches the frames whose own taps hold it
    and no others, an infinity as an infinity; one whose bfloat16 would be infinite is a number like any other."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] nonfinite short sr={sr} hop={hop} {n_bins} {B}x{L} {bad}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, n_taps=6144 if hop == 96 else 0, fmt=nb.NNA_OUT_COMPLEX,
                           device=0)
    assert nb.nna_plan_applied_tiles(plan, B, L)[1] == ((128, 2) if B == 400 else (64, 1))
    x = (0.3 * np.random.default_rng([47, hop, n_bins]).standard_normal((B, L))).astype(np.float32)
    b = B // 2
    x[b, at] = 0.0
    clean = nb.nna_cqt(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    x[b, at] = bad
    got = nb.nna_cqt(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(np.delete(got, b, 0), np.delete(clean, b, 0))
    got, clean = got[b].reshape(n_bins, 2, -1), clean[b].reshape(n_bins, 2, -1)
    kernels = np.stack(oracle.cqt_kernels(sr, fmin, n_bins, bpo, n_taps=plan.info()["taps"]), 1)
    half, lengths = kernels.shape[2] // 2, nb.nna_plan_cqt_lengths(plan)
    tap = half + at - hop * np.arange(got.shape[2])  # of the sample, in every frame; its mirror images lie outside these kernels
    assert lengths[-24] < min(at, L - at)
    for k in range(n_bins - 24, n_bins):
        s = half - (int(lengths[k]) + 1) // 2
        meets = (tap >= s) & (tap < s + int(lengths[k]))
        assert np.abs(got[k][:, ~meets] - clean[k][:, ~meets]).max(initial=0.0) <= 1e-5 * np.abs(clean).max(), k
        w = kernels[k][:, tap[meets]]
        if np.isfinite(bad):
            # the sample's products dwarf the others; two float32 roundings, of the tap and of the product
            assert np.abs(got[k][:, meets] - w * bad).max(initial=0.0) <= 2e-7 * np.abs(w).max(initial=0.0) * bad, k
        elif bad == bad:
            sure = np.abs(w) > 1e-6 * np.abs(w).max(initial=0.0)
            assert np.array_equal(got[k][:, meets][sure], (np.sign(w) * bad)[sure]), k
        else:
            assert np.isnan(got[k][:, meets]).all(), k
