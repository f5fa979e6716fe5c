"""Constant-Q kernels tap by tap: every form of the tiles, by whole hops and by the kernels' own taps, against the oracle; each case names the
form it runs.  Remainders of a tile, tiles across waveforms, one frame a waveform, columns past a row's last."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
# of the output's peak: float32 taps (2.6e-8 of a kernel's norm) and sums in blocks of 32 products (3e-7 at most)
TOL = 1e-6

CASES = [
    # sr, hop of octave 0, fmin, n_bins, bins per octave, octave, B, L, (form, frames, columns at a time, samples of a hop)
    (8000, 8, 400.0, 24, 12, 1, 120, 1203, (0, 64, 0, 4)),               # words of four, 64 frames
    (44100, 256, 520.0, 36, 36, 0, 140, 60001, (4, 64, 64, 256)),        # 64 frames by columns, kernels of 17 hops, two items
    (44100, 128, 260.0, 36, 36, 0, 70, 60001, (4, 64, 32, 128)),         # ... of 69
    (44100, 512, 800.0, 36, 36, 0, 130, 80003, (4, 64, 128, 512)),       # ... of seven, 128 columns at a time
    (22050, 1000, 250.0, 12, 12, 0, 3, 30001, (2, 16, 0, 1000)),         # 16 frames in a CU's LDS
    (22050, 512, 3100.0, 12, 12, 0, 300, 65537, (3, 128, 32, 128)),      # own taps: 128 frames
    (22050, 1024, 3100.0, 12, 12, 0, 60, 200003, (1, 32, 0, 128)),       # ... 32
    (22050, 512, 3100.0, 12, 12, 0, 2, 30001, (2, 16, 0, 128)),          # ... 16
    (44100, 512, 2600.0, 12, 12, 0, 270, 65537, (4, 64, 128, 320)),      # ... 64, 64 columns past the last
    (44100, 1000, 740.0, 12, 12, 0, 400, 100003, (4, 64, 128, 1024)),    # ... more than the hop
    (44100, 1500, 1000.0, 24, 24, 0, 3, 30002, (2, 15, 0, 1536)),        # ... in a CU's LDS
    (16000, 512, 1700.0, 36, 36, 0, 3, 30001, (2, 16, 0, 512)),          # two items of own taps that save too little
    (22050, 600, 3100.0, 36, 36, 0, 9, 30001, (2, 16, 0, 384)),          # two items, two widths
    (8000, 200, 800.0, 12, 12, 0, 90, 190, (2, 16, 0, 192)),             # a frame a waveform
]


def _octave(nb, sr, hop, fmin, n_bins, bpo, a):
    plan = nb.nna_plan_cqt2010v2(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, fmt=nb.NNA_OUT_COMPLEX, device=0)
    part = nb.nna_plan_part(plan, a)
    hi = n_bins - a * bpo
    lo = max(0, hi - bpo)
    return part, dict(sr=sr, hop=hop >> a, fmin=fmin * 2.0 ** ((lo + a * bpo) / bpo), n_bins=hi - lo, bins_per_octave=bpo,
                      n_taps=part.info()["taps"])


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[1] >> c[5]}-{c[3]}-{c[6]}x{c[7]}")
def test_form(case):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] short forms {case}", file=sys.stderr, flush=True)
    *args, B, L, tiles = case
    plan, cfg = _octave(nb, *args)
    assert nb.nna_plan_short_tiles(plan, B, L) == tiles
    x = (0.3 * np.random.default_rng([71, B, L]).standard_normal((B, L))).astype(np.float32)
    rows, T = nb.nna_out_shape(plan, B, L)
    out = torch.full((B, rows, T), float("nan"), device="cuda")
    got = nb.nna_cqt(plan, torch.from_numpy(x).cuda(), out=out)
    assert bool(torch.isfinite(got).all())
    some = sorted({0, B // 3, B // 2, B - 1})
    want = oracle.interleave(*oracle.cqt_complex(x[some], **cfg))
    got = got[some].cpu().numpy().astype(np.float64)
    for b in range(len(some)):
        assert np.abs(got[b] - want[b]).max() < TOL * np.abs(want[b]).max(), some[b]


@pytest.mark.parametrize("bad", [float("nan"), float("-inf"), 3.4e38])
@pytest.mark.parametrize("step", [1, 700])
@pytest.mark.parametrize("case", [CASES[0], CASES[1], CASES[6], CASES[8], CASES[12]], ids=lambda c: f"{c[1] >> c[5]}-{c[3]}-{c[6]}")
def test_samples_that_are_not_finite(case, step, bad):
    """Every sample of a stretch, or one in 700: frames whose own taps hold none are what they are without."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] short forms {case} {bad} every {step}", file=sys.stderr, flush=True)
    *args, B, L, tiles = case
    plan, cfg = _octave(nb, *args)
    x = (0.3 * np.random.default_rng([73, B, L]).standard_normal((B, L))).astype(np.float32)
    b = B // 2
    at = np.arange(L // 3, min(L, L // 3 + 900), step)
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
            hit = np.flatnonzero(mark[t * cfg["hop"] + s:t * cfg["hop"] + s + int(lengths[k])])
            if hit.size == 0:
                assert np.abs(got[k][:, t] - clean[k][:, t]).max() <= 1e-6 * np.abs(clean).max(), (k, t)
            elif np.isfinite(bad):
                # float32 sums of the products with large samples; the other samples' share is what was there without
                w = np.array([re[k][s + hit].sum(), im[k][s + hit].sum()]) * bad
                size = np.array([np.abs(re[k][s + hit]).sum(), np.abs(im[k][s + hit]).sum()]) * bad
                assert (np.abs(got[k][:, t] - w) <= 2e-5 * size + 2.0 * np.abs(clean).max()).all(), (k, t)
            elif (np.abs(re[k][s + hit]) > 1e-4 * np.abs(re[k]).max()).any():
                assert not np.isfinite(got[k][0, t]), (k, t)


BESIDE = [
    # sr, hop, fmin, n_bins, bins per octave, taps, B, L, frames and blocks of the kernels beside a basis, form of their tiles
    (22050, 512, 65.4, 84, 12, 0, 2, 100001, (64, 1), (4, 64, 128, 512)),
    (44100, 512, 65.4, 120, 24, 0, 260, 100000, (64, 1), (4, 64, 128, 512)),
    (16000, 96, 50.0, 60, 12, 6144, 3, 9003, (64, 1), (4, 64, 32, 96)),
    (22050, 512, 65.4, 84, 12, 131072, 1, 70001, (64, 1), (-1, 0, 0, 0)),   # kernels of more than 65,536 taps with their padding: none of these
    (8000, 64, 80.0, 60, 12, 0, 170, 9001, (128, 2), (-1, 0, 0, 0)),        # 128 frames, hop 64: items of two blocks a wave
]


@pytest.mark.parametrize("case", BESIDE, ids=lambda c: f"{c[1]}-{c[3]}-{c[5]}-{c[6]}x{c[7]}")
def test_beside_a_basis(case):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] short forms beside a basis {case}", file=sys.stderr, flush=True)
    sr, hop, fmin, n_bins, bpo, taps, B, L, direct, tiles = case
    cfg = dict(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, n_taps=taps)
    plan = nb.nna_plan_cqt(fmt=nb.NNA_OUT_COMPLEX, device=0, **cfg)
    assert nb.nna_plan_applied_tiles(plan, B, L)[1] == direct and nb.nna_plan_short_tiles(plan, B, L) == tiles
    x = (0.3 * np.random.default_rng([89, B, L]).standard_normal((B, L))).astype(np.float32)
    rows, T = nb.nna_out_shape(plan, B, L)
    out = torch.full((B, rows, T), float("nan"), device="cuda")
    got = nb.nna_cqt(plan, torch.from_numpy(x).cuda(), out=out)
    assert bool(torch.isfinite(got).all())
    some = sorted({0, B // 2, B - 1})
    want = oracle.interleave(*oracle.cqt_complex(x[some], **cfg))
    got = got[some].cpu().numpy().astype(np.float64)
    for b in range(len(some)):
        assert np.abs(got[b] - want[b]).max() < TOL * np.abs(want[b]).max(), some[b]


@pytest.mark.parametrize("seed", range(30))
def test_any_shape_against_the_general_kernel(seed):
    """Hops, taps, bins, lengths and batches of any kind: the octave against the same kernels made trainable, which run the general kernel.
    Its float32 chains are off by 3.3e-6 of the output's peak over 1,400 such cases."""
    import torch
    from paper_1912_12055_amd import binding as nb
    rng = np.random.default_rng([97, seed])
    sr, bpo = int(rng.choice([8000, 16000, 22050, 44100])), int(rng.choice([1, 3, 12, 17, 24, 36, 50]))
    hop = 4 * int(rng.choice([1, 2, 3, 5, 8, 9, 16, 24, 25, 32, 48, 64, 75, 125, 128, 150, 160, 250, 256, 375, 500]))
    n_bins, Q = int(rng.integers(1, bpo + 1)), 1.0 / (2.0 ** (1.0 / bpo) - 1.0)
    longest = int(2.05 * Q * 2.0 ** ((n_bins - 1) / bpo)) + int(rng.choice([1, 5, 30, 100, 300, 700, 1500]))
    taps = 2 * (longest // 2 + 1) + 2 * int(rng.integers(0, 200))
    L = max(taps // 2 + 1, (int(rng.choice([1, 2, 5, 20, 131, 345])) - 1) * hop) + int(rng.integers(0, hop)) + 4
    B = max(1, min(int(10.0 ** rng.uniform(0.0, 4.8)) // (1 + L // hop), 30000000 // L))
    cfg = dict(sr=sr, hop=hop, fmin=Q * sr / longest, n_bins=n_bins, bins_per_octave=bpo, n_taps=taps, fmt=nb.NNA_OUT_COMPLEX, device=0)
    plan = nb.nna_plan_part(nb.nna_plan_cqt2010v2(**cfg), 0)
    print(f"[case] short forms {cfg} {B}x{L} {nb.nna_plan_short_tiles(plan, B, L)}", file=sys.stderr, flush=True)
    x = torch.from_numpy(rng.standard_normal((B, L)).astype(np.float32)).cuda()
    rows, T = nb.nna_out_shape(plan, B, L)
    got = nb.nna_cqt(plan, x, out=torch.full((B, rows, T), float("nan"), device="cuda"))
    want = nb.nna_cqt(nb.nna_plan_trainable(nb.nna_plan_cqt(**cfg)), x)
    assert float((got - want).abs().max()) < 5e-6 * float(want.abs().max())
