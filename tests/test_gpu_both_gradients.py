"""Training steps that want both gradients of an STFT stage at once, in one launch or two, against the calls that want one
and against 64 bits."""
import sys

import pytest

pytestmark = pytest.mark.gpu


def _gradients_64(x, W, gout, hop):
    """Of complex output: the bank's and the waveform's gradient, in 64 bits."""
    import torch
    (B, L), K, T = x.shape, W.shape[1], gout.shape[2]
    at = torch.arange(T, device=x.device)[:, None] * hop + torch.arange(K, device=x.device) - K // 2
    at = at.abs()
    at = torch.where(at >= L, 2 * (L - 1) - at, at)
    gw, gx = torch.zeros(W.shape, dtype=torch.float64, device=x.device), torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    for b in range(B):
        g = gout[b].double()
        gw += g @ x[b].double()[at]
        gx[b].index_add_(0, at.reshape(-1), (g.T @ W.double()).reshape(-1))
    gw[[1, -1]] = 0  # the imaginary kernels of bins 0 and n_fft / 2 are zero and no parameters
    return gw, gx


# n_fft, hop, B, L: 256 + 176 tiles; a bank of few tiles in pieces beside a wave of few; more than one launch takes; one frame
@pytest.mark.parametrize("n_fft,hop,B,L", [(2048, 512, 16, 44217), (512, 160, 5, 9001), (1024, 256, 3, 5001), (512, 128, 120, 40001), (256, 256, 1, 129)])
def test_both_against_each(n_fft, hop, B, L):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] both gradients n_fft={n_fft} {B}x{L}", file=sys.stderr, flush=True)
    gen = torch.Generator().manual_seed(n_fft + B)
    plan = nb.nna_plan_trainable(nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=nb.NNA_OUT_POWER, device=0))
    x = torch.randn((B, L), generator=gen).cuda()
    gout = torch.randn(tuple(nb.nna_stft(plan, x).shape), generator=gen).cuda()
    gw, gx = nb.nna_stft_backward(plan, x, gout)
    # the same products, summed onto the output piece by piece in any order: up to 44 pieces, half an ulp of the running sum each
    for got, ref in ((gw, nb.nna_stft_backward(plan, x, gout, want_gx=False)[0]), (gx, nb.nna_stft_backward(plan, x, gout, want_gw=False)[1])):
        assert (got - ref).abs().max() <= 44 * 2.0 ** -24 * ref.abs().max()


# tiles of the waveform gradient in parts: 16 of one tile, of few, of kernels of many hops; hops that are no multiple of 128
@pytest.mark.parametrize("sr,hop,fmin,n_bins,bpo,B,L", [(8000, 128, 300.0, 5, 12, 1, 4001), (22050, 512, 65.4, 60, 12, 2, 30001), (16000, 256, 60.0, 84, 24, 3, 20000),
                                                        (16000, 96, 80.0, 30, 12, 2, 9000)])
def test_waveform_gradient_in_parts(sr, hop, fmin, n_bins, bpo, B, L):
    """A few waveforms' gradients against 64 bits and against a batch whose tiles are taken whole: the same products, added in up to 16 parts."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] waveform gradient in parts {sr} {hop} {n_bins} {B}x{L}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_trainable(nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, fmt=nb.NNA_OUT_COMPLEX, device=0))
    gen = torch.Generator().manual_seed(hop + L)
    L = max(L, plan.info()["taps"] // 2 + 3)
    x = torch.randn((B, L), generator=gen).cuda()
    gout = torch.randn(tuple(nb.nna_cqt(plan, x).shape), generator=gen).cuda()
    few = nb.nna_cqt_backward(plan, x, gout, want_gw=False)[1]
    # sums of up to 2 n_bins x 100 shifts in chains: a chain of n roundings is off by sqrt(n) 2^-24 of its terms' norm
    _, ref = _gradients_64(x, nb.nna_plan_get_bank(plan), gout, hop)
    assert (few - ref).abs().max() <= 2e-6 * ref.abs().max()
    n = 520 // B + 1
    many = nb.nna_cqt_backward(plan, x.repeat(n, 1), gout.repeat(n, 1, 1), want_gw=False)[1]
    assert (few - many[:B]).abs().max() <= 2e-6 * many.abs().max()
    assert (few - many[-B:]).abs().max() <= 2e-6 * many.abs().max()


# 256 + 176 tiles of 44 and 64 chunks; 16 + 440 of 440 and 16; 64 + 448 of 192 and 32; 6 + 378 of 504 and 8
@pytest.mark.parametrize("n_fft,hop,B,L", [(2048, 512, 16, 44217), (512, 128, 30, 60000), (1024, 256, 26, 60000), (256, 128, 52, 40001)])
def test_sums_as_short_as_alone(n_fft, hop, B, L):
    """Neither gradient's sums are longer than those of the call that wants it alone: no further from 64 bits."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] both gradients against 64 bits n_fft={n_fft} {B}x{L}", file=sys.stderr, flush=True)
    gen = torch.Generator().manual_seed(n_fft + B)
    plan = nb.nna_plan_trainable(nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=nb.NNA_OUT_COMPLEX, device=0))
    x = torch.randn((B, L), generator=gen).cuda()
    gout = torch.randn(tuple(nb.nna_stft(plan, x).shape), generator=gen).cuda()
    ref = _gradients_64(x, nb.nna_plan_get_bank(plan), gout, hop)
    both = nb.nna_stft_backward(plan, x, gout)
    alone = nb.nna_stft_backward(plan, x, gout, want_gx=False)[0], nb.nna_stft_backward(plan, x, gout, want_gw=False)[1]
    for k in range(2):
        far = [float((g.double() - ref[k]).norm() / ref[k].norm()) for g in (both[k], alone[k])]
        print(f"[error] {'gw' if k == 0 else 'gx'} both {far[0]:.3e} alone {far[1]:.3e}", file=sys.stderr, flush=True)
        # the same partial sums (of up to 176 x 2^-24 / sqrt(3) of their norm), added onto the output in any order: a tenth for that
        assert far[0] <= 1.1 * far[1] and far[1] < 2e-6


# 9 and 3 output tiles: a workgroup's share is one waveform
@pytest.mark.parametrize("n_fft,hop,n_mels,B,L", [(2048, 512, 128, 64, 110250), (512, 128, 64, 200, 40000)])
def test_filterbank_sums_of_one_waveform(n_fft, hop, n_mels, B, L):
    """The filterbank's gradient of a batch: every waveform's frames summed by themselves, no further from 64 bits than those sums and their addition."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] filterbank gradient against 64 bits n_fft={n_fft} {B}x{L}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_trainable(nb.nna_plan_mel(n_fft=n_fft, hop=hop, n_mels=n_mels, device=0))
    gen = torch.Generator().manual_seed(B)
    x = torch.randn((B, L), generator=gen).cuda()
    gout = torch.randn((B,) + tuple(nb.nna_out_shape(plan, B, L)), generator=gen).cuda()
    window = torch.hann_window(n_fft, dtype=torch.float64, device="cuda")
    ref, alone = 0, 0
    for b in range(B):
        padded = torch.nn.functional.pad(x[None, b:b + 1].double(), (n_fft // 2, n_fft // 2), mode="reflect")[0, 0]
        ref = ref + gout[b].double() @ torch.fft.rfft(padded.unfold(0, n_fft, hop) * window).abs().square()
        alone = alone + nb.nna_mel_backward(plan, x[b:b + 1], gout[b:b + 1], want_gw=False, want_gx=False)[0].double()
    batch, alone = (float((g.double() - ref).norm() / ref.norm()) for g in (nb.nna_mel_backward(plan, x, gout, want_gx=False)[0], alone))
    print(f"[error] batch {batch:.3e} one by one {alone:.3e}", file=sys.stderr, flush=True)
    # adding B sums one after the other: a rounding of up to 2^-24 (a third of that squared on average) of what has been added, i / B of the whole squared
    assert batch ** 2 <= alone ** 2 + 2.0 ** -48 * B / 6 and batch < 2e-6
