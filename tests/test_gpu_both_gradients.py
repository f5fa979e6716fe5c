"""Training steps that want both gradients of an STFT stage at once, in one launch (uncut, in pieces) or two, against the calls that want one."""
import sys

import pytest

pytestmark = pytest.mark.gpu


# n_fft, hop, B, L: 256 + 176 tiles uncut; a bank of few tiles in pieces beside a wave of few; more than one launch takes; one frame
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
