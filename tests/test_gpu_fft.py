"""The STFT and Mel layers' fast Fourier transform against the oracle, at the sizes where it can go wrong: every kernel of
its own (N = 64 .. 4,096), the general kernel (odd half lengths, each radix, the largest that fits; 66 has a factor of 11 and stays a contraction), ragged hops, frames
that reach into both mirrored ends, tiles that span waveforms, a single frame, filters at both ends of the spectrum."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
# Relative to each output's peak.  A transform of N points in float32 accumulates about log2(N) roundings of 2^-24 per
# value, a bin at most sqrt(N) of them relative to the peak of a tone: 1e-6 at 13 stages; ten times that is asserted.
TOL = 1e-5


@pytest.fixture(scope="module")
def nb():
    from paper_1912_12055_amd import binding
    binding.lib()
    return binding


def _wave(seed, B, L):
    rng = np.random.default_rng([19, seed])
    t = np.arange(L)
    x = 0.1 * rng.standard_normal((B, L))
    for b in range(B):
        x[b] += rng.uniform(0.1, 0.5) * np.sin(2 * np.pi * rng.uniform(0.01, 0.45) * t + rng.uniform(0, 6.28))
    return x.astype(np.float32)


def _err(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    assert got.shape == ref.shape and np.all(np.isfinite(got))
    return max(np.abs(got[b] - ref[b]).max() / np.abs(ref[b]).max() for b in range(ref.shape[0]))


# n_fft, hop, B, L, center
CASES = [
    (64, 16, 3, 1000, True), (128, 100, 2, 3001, True), (256, 64, 37, 700, True), (512, 160, 3, 9001, False),
    (1024, 256, 2, 20011, True), (2048, 512, 5, 22050, True), (2048, 441, 1, 2048, False), (4096, 512, 3, 9999, True),
    (4096, 1024, 2, 4096, False), (2048, 3, 1, 1200, True),
    (66, 11, 2, 500, True), (70, 35, 5, 200, True), (98, 24, 2, 400, True), (90, 45, 2, 333, False),
    (400, 160, 4, 16001, True), (882, 441, 2, 8000, True), (768, 192, 3, 5000, True), (3000, 750, 2, 9000, True),
    (8192, 2048, 2, 30000, True), (12000, 3000, 1, 30000, True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}-hop{c[1]}-{c[2]}x{c[3]}{'' if c[4] else '-nocenter'}")
def test_every_output_format(nb, case):
    n_fft, hop, B, L, center = case
    print(f"[case] fft {case}", file=sys.stderr, flush=True)
    import torch
    x = _wave(n_fft + hop, B, L)
    xd = torch.from_numpy(x).to("cuda:0")
    kw = dict(n_fft=n_fft, hop=hop, center=center)
    re, im = oracle.stft_complex(x, window=oracle.WIN_HANN, **kw)
    power = re * re + im * im
    plan = lambda fmt: nb.nna_plan_stft(win=nb.NNA_WIN_HANN, fmt=fmt, device=0, **kw)
    assert _err(nb.nna_stft(plan(nb.NNA_OUT_MAGNITUDE), xd), np.sqrt(power)) < TOL
    assert _err(nb.nna_stft(plan(nb.NNA_OUT_POWER), xd), power) < TOL
    assert _err(nb.nna_stft(plan(nb.NNA_OUT_COMPLEX), xd), oracle.interleave(re, im)) < TOL
    keep = power > 1e-6 * power.max()
    # absolute error 1e-5 of the peak magnitude on a bin 1e-3 of it: 1e-2 relative, 2e-2 in the logarithm of the power
    log = nb.nna_stft(plan(nb.NNA_OUT_LOG), xd).cpu().numpy()
    assert np.abs(log - np.log(np.maximum(power, 1e-10)))[keep].max() < 2e-2
    d = nb.nna_stft(plan(nb.NNA_OUT_PHASE), xd).cpu().numpy() - np.arctan2(im, re)
    assert np.abs((d + np.pi) % (2 * np.pi) - np.pi)[keep].max() < 1e-2


@pytest.mark.parametrize("n_fft,hop,B,L,n_mels,power", [
    (2048, 512, 3, 22050, 128, 2.0), (4096, 512, 2, 20000, 512, 2.0), (1024, 256, 20, 3000, 1, 1.0), (512, 160, 2, 9001, 40, 1.0),
    (256, 64, 5, 4000, 300, 2.0), (400, 160, 3, 16000, 80, 2.0), (64, 32, 2, 500, 7, 2.0), (126, 63, 2, 900, 9, 1.0)])
def test_mel_bands_and_their_spectrogram(nb, n_fft, hop, B, L, n_mels, power):
    print(f"[case] fft mel n_fft={n_fft} hop={hop} B={B} L={L} n_mels={n_mels}", file=sys.stderr, flush=True)
    import torch
    x = _wave(n_fft + n_mels, B, L)
    xd = torch.from_numpy(x).to("cuda:0")
    ref = oracle.mel(x, sr=22050, n_fft=n_fft, hop=hop, n_mels=n_mels, power=power)
    plan = nb.nna_plan_mel(sr=22050, n_fft=n_fft, hop=hop, n_mels=n_mels, power=power, device=0)
    assert _err(nb.nna_mel(plan, xd), ref) < TOL
    mel, spec = nb.nna_mel_with_stft(plan, xd)
    assert _err(mel, ref) < TOL
    fmt = oracle.POWER if power == 2.0 else oracle.MAGNITUDE
    assert _err(spec, oracle.stft(x, n_fft=n_fft, hop=hop, fmt=fmt)) < TOL


# one frame in twenty reaches past an end, and more: the same frames from either launch
@pytest.mark.parametrize("n_fft", [64, 256, 1024, 2048, 4096])
@pytest.mark.parametrize("kind", ["POWER", "COMPLEX", "MEL"])
def test_frames_at_the_ends_few_or_many(nb, n_fft, kind):
    import torch
    print(f"[case] fft ends {n_fft} {kind}", file=sys.stderr, flush=True)
    hop = n_fft // 4
    L = {T: (T - 1) * hop for T in (79, 80)}  # four frames reach past an end
    x = torch.from_numpy(_wave(n_fft, 3, L[80])).to("cuda:0")
    if kind == "MEL":
        plan = nb.nna_plan_mel(n_fft=n_fft, hop=hop, n_mels=12, device=0)
    else:
        plan = nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=getattr(nb, "NNA_OUT_" + kind), device=0)
    run = nb.nna_mel if kind == "MEL" else nb.nna_stft
    few, many = run(plan, x), run(plan, x[:, :L[79]].contiguous())
    assert few.shape[2] == 80 and many.shape[2] == 79
    assert torch.equal(few[:, :, :77], many[:, :, :77])
    if kind == "POWER":
        ref = oracle.stft_complex(x[:, :L[79]].cpu().numpy(), n_fft=n_fft, hop=hop, window=oracle.WIN_HANN)
        assert _err(many, ref[0] ** 2 + ref[1] ** 2) < TOL
