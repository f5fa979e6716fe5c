"""Constant-Q kernels tap by tap: samples next to the largest float32 number, a few of which are no bfloat16 (their products are added one by
one), among others that are: the sums are the float32 sums, and the same at every call."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CASES = [
    # sr, hop, fmin, n_bins, bins per octave, B, L
    (8000, 4, 400.0, 12, 12, 1, 2001),
    (22050, 64, 1000.0, 24, 24, 300, 9002),
    (22050, 512, 3100.0, 12, 12, 300, 65537),
    (44100, 256, 520.0, 36, 36, 140, 60001),
]


def _plan(sr, hop, fmin, n_bins, bpo):
    from paper_1912_12055_amd import binding as nb
    plan = nb.nna_plan_part(nb.nna_plan_cqt2010v2(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, fmt=nb.NNA_OUT_COMPLEX, device=0), 0)
    assert nb.nna_plan_short_tiles(plan, 1, 30 * hop + plan.info()["taps"])[0] >= 0
    return nb, plan


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[1]}-{c[3]}-{c[5]}x{c[6]}")
@pytest.mark.parametrize("among", [0.3, 3.38e38], ids=["noise", "large"])
def test_large_samples(case, among):
    import torch
    *args, B, L = case
    nb, plan = _plan(*args)
    print(f"[case] short kernels, large samples {case} among {among}", file=sys.stderr, flush=True)
    rng = np.random.default_rng([79, B, L])
    x = np.float32(0.3) * rng.standard_normal((B, L)).astype(np.float32)
    b, taps = B // 2, plan.info()["taps"]
    re, im = oracle.cqt_kernels(args[0], args[2], args[3], args[4], n_taps=taps)
    # signs of a kernel of one frame in the middle: its sums are as large as they can be
    t = (L // 2 // args[1])
    k = args[3] // 2
    span = np.arange(taps) + t * args[1] - taps // 2
    inside = (span >= 0) & (span < L) & (re[k] != 0.0)
    sign = np.where(re[k] < 0.0, -1.0, 1.0)[inside]
    x[b, span[inside]] = np.abs(x[b, span[inside]]) * sign if among < 1 else among * sign
    few = rng.choice(np.flatnonzero(inside), 40, replace=False)
    x[b, span[few]] = 3.4e38 * np.sign(np.where(re[k][few] < 0.0, -1.0, 1.0)) * rng.uniform(0.9985, 1.0, 40)
    x = x.astype(np.float32)
    assert np.isfinite(x).all()
    xd = torch.from_numpy(x).cuda()
    first = nb.nna_cqt(plan, xd)
    for _ in range(8):
        assert int((nb.nna_cqt(plan, xd) != first).sum()) == 0
    got = first[b].cpu().numpy().astype(np.float64)
    want = oracle.interleave(*oracle.cqt_complex(x[b:b + 1], hop=args[1], sr=args[0], fmin=args[2], n_bins=args[3], bins_per_octave=args[4], n_taps=taps))[0]
    assert np.isfinite(got).all()
    # float32 sums in blocks of 32, and chains of up to forty products added to them
    assert np.abs(got - want).max() < 4e-6 * np.abs(want).max()


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[1]}-{c[3]}-{c[5]}x{c[6]}")
@pytest.mark.parametrize("exponent", [-118, -110, -100, 0, 100, 118, 124])
def test_range(case, exponent):
    """Samples of every magnitude: three bfloat16 of 2^10 times a sample hold it from 2^-120 up to 2^118, larger ones are added one by one.
    A bin's error, 2-norm: 0.8e-7 .. 2.6e-7 measured; the float32 instruction's chains 4e-7 .. 9e-6."""
    import torch
    *args, B, L = case
    nb, plan = _plan(*args)
    print(f"[case] short kernels, range {case} 2^{exponent}", file=sys.stderr, flush=True)
    x = (0.3 * np.random.default_rng([83, B, L]).standard_normal((B, L))).astype(np.float32)
    got = nb.nna_cqt(plan, torch.from_numpy(np.ldexp(x, exponent)).cuda())[[0, B // 2, B - 1]].cpu().numpy()
    got = np.ldexp(got.astype(np.float64), -exponent)
    # (at 2^-118 samples are rounded to the least float32 numbers: those that were put in)
    x = np.ldexp(np.ldexp(x[[0, B // 2, B - 1]], exponent).astype(np.float64), -exponent).astype(np.float32)
    want = oracle.interleave(*oracle.cqt_complex(x, hop=args[1], sr=args[0], fmin=args[2], n_bins=args[3], bins_per_octave=args[4],
                                                 n_taps=plan.info()["taps"]))
    for b in range(3):
        err, ref = (got[b] - want[b]).reshape(args[3], -1), want[b].reshape(args[3], -1)
        rel = np.linalg.norm(err, axis=1) / np.linalg.norm(ref, axis=1)
        assert rel.max() < 4.5e-7, (b, rel.argmax(), rel.max())
