"""Constant-Q kernels tap by tap on the bfloat16 matrix pipe: the octaves of the downsampling plans, one by one against the oracle.  Hops
of 4 (words of four samples in LDS), of 8 and more, of whole 32 columns; batches that reach tiles of 16, 32, 64 and 128 frames
(tests/test_gpu_short_forms.py names the tiles of its cases); tiles that span waveforms, one and several items, ends inside a run of four samples; samples that are not finite, few and many."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
# of the output's peak: float32 taps (2.6e-8 of a kernel's norm) and sums in blocks of 32 products (3e-7 at most)
TOL = 1e-6

CASES = [
    # sr, hop of octave 0, fmin, n_bins, bins per octave, octave, B, L
    (8000, 8, 400.0, 24, 12, 1, 3, 2001),         # hop 4, 16 frames a tile
    (8000, 8, 400.0, 24, 12, 1, 60, 1203),        # ... of 32, across waveforms
    (8000, 8, 400.0, 24, 12, 0, 9, 8005),         # hop 8, 32 frames
    (8000, 24, 400.0, 60, 30, 1, 7, 4003),        # hop 12, two items of a plan, the second of six bins
    (16000, 96, 500.0, 20, 12, 0, 40, 9001),      # a hop that is no power of two
    (22050, 64, 1000.0, 24, 24, 0, 300, 9002),    # hop 64, 64 frames
    (22050, 512, 1000.0, 12, 12, 0, 2, 30001),    # hop 512, 16 frames
    (22050, 256, 1500.0, 24, 24, 0, 1900, 9003),  # columns
    (22050, 512, 700.0, 20, 12, 0, 900, 37001),   # columns, kernels of less than a hop
]


def _octave(nb, sr, hop, fmin, n_bins, bpo, a):
    plan = nb.nna_plan_cqt2010v2(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, fmt=nb.NNA_OUT_COMPLEX, device=0)
    part = nb.nna_plan_part(plan, a)
    hi = n_bins - a * bpo
    lo = max(0, hi - bpo)
    return part, dict(sr=sr, hop=hop >> a, fmin=fmin * 2.0 ** ((lo + a * bpo) / bpo), n_bins=hi - lo, bins_per_octave=bpo,
                      n_taps=part.info()["taps"])


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[1] >> c[5]}-{c[3]}-{c[6]}x{c[7]}")
def test_octave(case):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] short kernels {case}", file=sys.stderr, flush=True)
    *args, B, L = case
    plan, cfg = _octave(nb, *args)
    x = (0.3 * np.random.default_rng([53, B, L]).standard_normal((B, L))).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    rows, T = nb.nna_out_shape(plan, B, L)
    out = torch.full((B, rows, T), float("nan"), device="cuda")
    got = nb.nna_cqt(plan, xd, out=out)
    assert bool(torch.isfinite(got).all())
    some = sorted({0, B // 3, B // 2, B - 1})
    want = oracle.interleave(*oracle.cqt_complex(x[some], **cfg))
    got = got[some].cpu().numpy().astype(np.float64)
    for b in range(len(some)):
        assert np.abs(got[b] - want[b]).max() < TOL * np.abs(want[b]).max(), some[b]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3.4e38])
@pytest.mark.parametrize("step", [1, 700])
@pytest.mark.parametrize("case", [CASES[1], CASES[5], CASES[6], CASES[7]], ids=lambda c: f"{c[1] >> c[5]}-{c[6]}")
def test_samples_that_are_not_finite(case, step, bad):
    """Every sample of a stretch, or one in 700: frames whose own taps hold none are what they are without; a number above the largest
    bfloat16 is one like any other."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] short kernels {case} {bad} every {step}", file=sys.stderr, flush=True)
    *args, B, L = case
    plan, cfg = _octave(nb, *args)
    x = (0.3 * np.random.default_rng([59, B, L]).standard_normal((B, L))).astype(np.float32)
    b = B // 2
    at = np.arange(L // 3, L // 3 + 900, step)
    at = at[at < L]
    x[b, at] = 0.0
    clean = nb.nna_cqt(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    x[b, at] = bad
    got = nb.nna_cqt(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(np.delete(got, b, 0), np.delete(clean, b, 0))
    re, im = oracle.cqt_kernels(cfg["sr"], cfg["fmin"], cfg["n_bins"], cfg["bins_per_octave"], n_taps=cfg["n_taps"])
    lengths, half = nb.nna_plan_cqt_lengths(plan), re.shape[1] // 2
    got, clean = got[b].reshape(cfg["n_bins"], 2, -1), clean[b].reshape(cfg["n_bins"], 2, -1)
    mark = np.zeros(L, bool)
    mark[at] = True
    mark = np.pad(mark, half, mode="reflect")
    for k in range(cfg["n_bins"]):
        s = half - (int(lengths[k]) + 1) // 2
        for t in range(got.shape[2]):
            first = t * cfg["hop"] + s
            hit = np.flatnonzero(mark[first:first + int(lengths[k])])
            if hit.size == 0:
                assert np.abs(got[k][:, t] - clean[k][:, t]).max() <= 1e-6 * np.abs(clean).max(), (k, t)
            elif np.isfinite(bad):
                # sums of up to 900 float32 products; the other samples' share is what was there without
                w = np.array([re[k][s + hit].sum(), im[k][s + hit].sum()]) * bad
                size = np.array([np.abs(re[k][s + hit]).sum(), np.abs(im[k][s + hit]).sum()]) * bad
                assert (np.abs(got[k][:, t] - w) <= 2e-5 * size + 2.0 * np.abs(clean).max()).all(), (k, t)
            elif (np.abs(re[k][s + hit]) > 1e-4 * np.abs(re[k]).max()).any():
                assert not np.isfinite(got[k][0, t]), (k, t)


@pytest.mark.parametrize("sr,hop,n_bins,bpo,B,L,blocks", [
    (22050, 512, 84, 12, 2, 100001, 1),      # beside hop-block items of 64, 128 and 256 frames
    (22050, 512, 83, 12, 200, 60003, 2),      # a last item of eleven bins
    (44100, 512, 120, 24, 260, 100000, 4),
    (16000, 96, 60, 12, 3, 9003, 1),         # 32 columns at a time
    (8000, 64, 60, 12, 4, 9002, 1),          # 64
])
def test_beside_hop_blocks(sr, hop, n_bins, bpo, B, L, blocks):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] short kernels beside hop-blocks sr={sr} hop={hop} n_bins={n_bins} {B}x{L}", file=sys.stderr, flush=True)
    cfg = dict(sr=sr, hop=hop, fmin=50.0 if hop == 96 else 80.0 if hop == 64 else 65.4, n_bins=n_bins, bins_per_octave=bpo,
               n_taps=6144 if hop == 96 else 0)
    plan = nb.nna_plan_cqt(fmt=nb.NNA_OUT_COMPLEX, device=0, **cfg)
    tiles = nb.nna_plan_applied_tiles(plan, B, L)
    assert tiles[0][1] == blocks and tiles[1] == (64, 1)
    x = (0.3 * np.random.default_rng([61, B, L]).standard_normal((B, L))).astype(np.float32)
    rows, T = nb.nna_out_shape(plan, B, L)
    out = torch.full((B, rows, T), float("nan"), device="cuda")
    got = nb.nna_cqt(plan, torch.from_numpy(x).cuda(), out=out)
    assert bool(torch.isfinite(got).all())
    some = sorted({0, B // 2, B - 1})
    got = got[some].cpu().numpy().astype(np.float64)
    want = oracle.interleave(*oracle.cqt_complex(x[some], **cfg))
    for b in range(len(some)):
        assert np.abs(got[b] - want[b]).max() < TOL * np.abs(want[b]).max(), some[b]
