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
