"""STFT and Mel plans below 256 samples, whose fast Fourier transform gives way to the contraction on large batches: both forms
against the oracle, on the same waveforms alone and repeated past the line."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
TOL = 1e-5  # of the peak, as for either form by itself


def _err(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    return np.abs(got - ref).max() / np.abs(ref).max()


@pytest.mark.parametrize("n_fft,hop,frames", [(70, 17, 8300), (96, 32, 8300), (126, 63, 8300), (128, 32, 17000), (128, 50, 17000), (160, 40, 17000),
                                              (192, 32, 17000), (210, 105, 140000), (252, 63, 140000)])
def test_both_sides_of_the_line(n_fft, hop, frames):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fft line n_fft={n_fft} hop={hop}", file=sys.stderr, flush=True)
    L = 40 * hop + 11
    x = (0.3 * np.random.default_rng([47, n_fft]).standard_normal((3, L))).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    many = xd.repeat(frames // (3 * (1 + L // hop)) + 1, 1)
    re, im = oracle.stft_complex(x, n_fft=n_fft, hop=hop)
    for fmt, ref in ((nb.NNA_OUT_MAGNITUDE, np.hypot(re, im)), (nb.NNA_OUT_POWER, re * re + im * im), (nb.NNA_OUT_COMPLEX, oracle.interleave(re, im))):
        plan = nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=fmt, device=0)
        assert _err(nb.nna_stft(plan, xd), ref) < TOL
        out = nb.nna_stft(plan, many)
        assert _err(out[:3], ref) < TOL and _err(out[-3:], ref) < TOL
    ref = oracle.mel(x, n_fft=n_fft, hop=hop, n_mels=20)
    plan = nb.nna_plan_mel(n_fft=n_fft, hop=hop, n_mels=20, device=0)
    for batch in (xd, many):
        mel, spec = nb.nna_mel_with_stft(plan, batch)
        assert _err(nb.nna_mel(plan, batch)[-3:], ref) < TOL and _err(mel[-3:], ref) < TOL and _err(spec[-3:], re * re + im * im) < TOL
