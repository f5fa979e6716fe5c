"""The trainable STFT layer's three contractions (each float32 as three bfloat16) against the same sums in 64 bits: frame counts
around a tile, taps that are no multiple of a chunk, odd hops and lengths, samples and kernels of very different magnitudes."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
# six of the nine partial products: 2^-26 of each product dropped, float32 accumulation over n <= 2,048 terms; as the float32
# instruction, below 2e-6 of the result's norm
TOL = 4e-6


@pytest.mark.parametrize("n_fft,hop,B,L", [(64, 16, 1, 2032), (64, 16, 1, 2048), (400, 163, 3, 7001), (1024, 100, 2, 1999),
                                           (2048, 512, 5, 22050), (256, 256, 1, 129)])
@pytest.mark.parametrize("scale", [1.0, 1e-12])
def test_trainable_stft_power(n_fft, hop, B, L, scale):
    import torch
    from paper_1912_12055_amd import layers
    print(f"[case] split stft n_fft={n_fft} hop={hop} B={B} L={L} scale={scale}", file=sys.stderr, flush=True)
    gen = torch.Generator().manual_seed(n_fft + hop)
    x = torch.randn(B, L, generator=gen) * scale
    x[:, : L // 2] *= 1e-3
    layer = layers.STFT(n_fft=n_fft, hop_length=hop, sr=16000, output_format="Power", trainable=True)
    xd = x.cuda().requires_grad_(True)
    out = layer(xd)
    gout = torch.randn(out.shape, generator=gen)
    gw, gx = torch.autograd.grad(out, [layer.wsin_wcos, xd], gout.cuda())
    x64 = x.double().requires_grad_(True)
    w64 = layer.wsin_wcos.detach().cpu().double().requires_grad_(True)
    frames = torch.nn.functional.pad(x64[:, None], (n_fft // 2, n_fft // 2), mode="reflect")[:, 0].unfold(1, n_fft, hop)
    c = frames @ w64.t()
    ref = (c[..., 0::2] ** 2 + c[..., 1::2] ** 2).transpose(1, 2)
    rw, rx = torch.autograd.grad(ref, [w64, x64], gout.double())
    for name, got, want in (("out", out, ref), ("gw", gw, rw), ("gx", gx, rx)):
        got, want = got.detach().cpu().double().numpy(), want.detach().numpy()
        assert np.linalg.norm(got - want) < TOL * np.linalg.norm(want), name


@pytest.mark.parametrize("scale", [1e-30, 1e30])
def test_trainable_stft_range(scale):
    """Three bfloat16 hold a float32 from 2^-110 up to where its neighbour would be infinite: no more is lost at 1e-30 or 1e30 than
    at 1, forward and for the kernels' gradient (complex output, so that nothing is squared)."""
    import torch
    from paper_1912_12055_amd import layers
    n_fft, hop, B, L = 512, 128, 3, 9001
    print(f"[case] split stft range scale={scale}", file=sys.stderr, flush=True)
    gen = torch.Generator().manual_seed(7)
    x = torch.randn(B, L, generator=gen) * scale
    layer = layers.STFT(n_fft=n_fft, hop_length=hop, sr=16000, output_format="Complex", trainable=True)
    out = layer(x.cuda())
    gout = torch.randn(out.shape, generator=gen)
    (gw,) = torch.autograd.grad(out, [layer.wsin_wcos], gout.cuda())
    w64 = layer.wsin_wcos.detach().cpu().double().requires_grad_(True)
    frames = torch.nn.functional.pad(x.double()[:, None], (n_fft // 2, n_fft // 2), mode="reflect")[:, 0].unfold(1, n_fft, hop)
    c = (frames @ w64.t()).transpose(1, 2)
    (rw,) = torch.autograd.grad(c, [w64], gout.double())
    rw[[1, n_fft + 1]] = 0.0  # the sine kernels of k = 0 and n_fft / 2 vanish: no parameters
    for name, got, want in (("out", out, c), ("gw", gw, rw)):
        got, want = got.detach().cpu().double().numpy().ravel(), want.detach().numpy().ravel()
        assert np.linalg.norm(got - want) < TOL * np.linalg.norm(want), name


@pytest.mark.parametrize("fmt", ["MAGNITUDE", "COMPLEX"])
def test_short_and_large_batches_agree(fmt):
    """A short batch's workgroups take half the rows of a large one's, and its waveform gradient is summed in pieces: the same sums in the
    same order forwards, the same sums backwards."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] split short and large {fmt}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_trainable(nb.nna_plan_stft(n_fft=1024, hop=256, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0))
    gen = torch.Generator().manual_seed(67)
    x = torch.randn((40, 60001), generator=gen).cuda()  # 74 x 8 tiles of 128 x 128; five of them: 10 x 8
    out = nb.nna_stft(plan, x)
    few = nb.nna_stft(plan, x[:5].contiguous())
    assert torch.equal(out[:5], few)
    gout = torch.randn(out.shape, generator=gen).cuda()
    _, gx = nb.nna_stft_backward(plan, x, gout)
    _, gx_few = nb.nna_stft_backward(plan, x[:5].contiguous(), gout[:5].contiguous())
    # sums of up to four frames, each in up to two pieces: float32 rounding of a few of them
    assert (gx[:5] - gx_few).norm() <= 2e-6 * gx_few.norm()
