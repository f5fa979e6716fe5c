"""Error of the constant-Q calls against 64 bits, bin by bin: sums are taken in short blocks, each rounded into a total."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
# Sums of m roundings with random partial sums are off by 2.5e-8 sqrt(m / 2) of their value: 2.8e-7 for a hop's 512 products (two a
# rounding) in one chain, 5.6e-7 and more for a whole kernel's 2,000.  Blocks of 32 products measure 1.7e-7 .. 3.0e-7 over every bin of
# these plans (2.3e-7 .. 3.9e-7 with the float32 instruction); one chain per bin 6.7e-7 .. 9.1e-7.
TOL = 4.5e-7


@pytest.mark.parametrize("kind,sr,hop,n_bins,bpo", [("cqt", 22050, 512, 84, 12), ("cqt", 44100, 512, 168, 24), ("cqt", 16000, 256, 84, 12),
                                                    ("cqt", 22050, 256, 120, 24), ("cqt1992", 16000, 256, 60, 12)])
def test_every_bin(kind, sr, hop, n_bins, bpo):
    _check(kind, sr, hop, n_bins, bpo, 1.0)


@pytest.mark.parametrize("kind,sr,hop,n_bins,bpo", [("cqt", 22050, 512, 84, 12), ("cqt1992", 16000, 256, 60, 12)])
@pytest.mark.parametrize("scale", [2.0 ** -100, 2.0 ** 100])
def test_range(kind, sr, hop, n_bins, bpo, scale):
    """Three bfloat16 hold samples, coordinates and weights as float32 does from 2^-110 up (measured: 2.0e-7 of a bin's norm from 1e-32 to
    3e37, 2e-6 at 1e-34, 2e-4 at 1e-36)."""
    _check(kind, sr, hop, n_bins, bpo, scale)


def _check(kind, sr, hop, n_bins, bpo, scale):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] cqt error {kind} sr={sr} hop={hop} n_bins={n_bins} scale={scale}", file=sys.stderr, flush=True)
    cfg = dict(sr=sr, hop=hop, fmin=32.7, n_bins=n_bins, bins_per_octave=bpo)
    make, run = (nb.nna_plan_cqt, nb.nna_cqt) if kind == "cqt" else (nb.nna_plan_cqt1992, nb.nna_cqt1992)
    plan = make(fmt=nb.NNA_OUT_COMPLEX, device=0, **cfg)
    assert nb.nna_plan_applied_tiles(plan, 1, 3 * plan.info()["taps"] // 2)[0][0] > 0
    x = (0.3 * np.random.default_rng([41, hop, n_bins]).standard_normal((1, 3 * plan.info()["taps"] // 2))).astype(np.float32)
    got = run(plan, torch.from_numpy(x * np.float32(scale)).cuda()).cpu().numpy().astype(np.float64)[0] / scale
    if kind == "cqt":
        re, im = oracle.cqt_complex(x, **cfg)
        want = oracle.interleave(re, im)[0]
    else:
        W = nb.nna_plan_applied_kernels(plan)  # (the oracle's two stages round nothing either, but have no complex output)
        K = W.shape[1]
        padded = np.pad(x[0].astype(np.float64), K // 2, mode="reflect")
        want = W @ np.stack([padded[t:t + K] for t in range(0, padded.size - K + 1, hop)], 1)
    err = (got - want).reshape(n_bins, -1)
    rel = np.linalg.norm(err, axis=1) / np.linalg.norm(want.reshape(n_bins, -1), axis=1)
    assert rel.max() < TOL, (rel.argmax(), rel.max())
