"""Trainable Mel layer: the filterbank's product takes frames of the whole batch in tiles that span waveforms.  Batches of one frame a
waveform to more than a tile of them, every waveform bit for bit what it is alone, and the fused kernel's result to rounding."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L", [(300, 30), (131, 61), (67, 100), (43, 259), (5, 4060), (3, 4100), (1, 9001)])
@pytest.mark.parametrize("n_mels", [1, 40, 130])
def test_batches_of_short_waveforms(B, L, n_mels):
    import torch
    from paper_1912_12055_amd import layers, binding as nb
    print(f"[case] mel product {B}x{L} n_mels={n_mels}", file=sys.stderr, flush=True)
    layer = layers.MelSpectrogram(sr=16000, n_fft=58, hop_length=32, n_mels=n_mels, trainable_mel=True, trainable_STFT=True)
    gen = torch.Generator().manual_seed(B + n_mels)
    with torch.no_grad():
        layer.mel_basis.copy_(torch.randn(layer.mel_basis.shape, generator=gen))
    x = torch.randn((B, L), generator=gen).cuda()
    with torch.no_grad():
        out = layer(x)
        for b in {0, B // 2, B - 1}:
            assert torch.equal(out[b], layer(x[b])[0])
    fused = nb.nna_mel(layer.plan, x)
    # sums of 30 float32 powers with weights of either sign: 30 roundings of 2^-24 of the largest terms, both ways
    assert (out - fused).abs().max() < 1e-5 * fused.abs().max()
    # the backward pass's product, gradient to the spectrogram, over the same tiles: linear in the upstream gradient
    g = torch.randn(out.shape, generator=torch.Generator().manual_seed(3)).cuda()
    xr = x.clone().requires_grad_(True)
    gx, = torch.autograd.grad(layer(xr), xr, g)
    one = x[B - 1:].clone().requires_grad_(True)
    g1, = torch.autograd.grad(layer(one), one, g[B - 1:])
    assert (gx[B - 1:] - g1).abs().max() <= 1e-5 * g1.abs().max()  # (the adds of the waveform gradient have no fixed order)


def test_forward_holds_a_bounded_spectrogram():
    import torch
    from paper_1912_12055_amd import layers
    print("[case] mel product memory", file=sys.stderr, flush=True)
    layer = layers.MelSpectrogram(sr=22050, n_fft=2048, hop_length=512, n_mels=40, trainable_mel=True)
    x = torch.randn((14000, 22050), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")  # 2.5 GB of spectrogram
    with torch.no_grad():
        layer(x[:4])
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        out = layer(x)
        assert torch.cuda.max_memory_allocated() - before < (1 << 30) + out.numel() * 4 + (64 << 20)
        for b in (0, 5937, 5938, 13999):
            assert torch.equal(out[b], layer(x[b])[0])
