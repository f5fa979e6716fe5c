"""Training steps whose forward pass keeps C: the same output bit for bit and the same gradients as the calls that compute C again."""
import sys

import pytest

pytestmark = pytest.mark.gpu
# partial sums meet in memory by atomic adds, in any order: float32 rounding of a few of them
TOL = 2e-6


def _close(got, want):
    assert (got is None) == (want is None)
    assert got is None or (got - want).norm() <= TOL * want.norm()


PLANS = [("stft", "POWER"), ("mel", "POWER"), ("cqt", "MAGNITUDE"), ("cqt", "POWER"), ("cqt", "LOG"), ("cqt", "PHASE")]


# frames short of, at and past a block of 32; waveforms that end inside a run of four samples; many frames
@pytest.mark.parametrize("B,L", [(1, 2100), (3, 4097), (2, 7003), (60, 9001)])
@pytest.mark.parametrize("kind,fmt", PLANS)
def test_same_as_recomputed(kind, fmt, B, L):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] kept {kind} {fmt} {B}x{L}", file=sys.stderr, flush=True)
    made = {"stft": lambda: nb.nna_plan_stft(n_fft=400, hop=100, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0),
            "mel": lambda: nb.nna_plan_mel(sr=16000, n_fft=512, hop=128, n_mels=40, device=0),
            "cqt": lambda: nb.nna_plan_cqt(sr=8000, hop=32, fmin=80.0, n_bins=31, bins_per_octave=12, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0)}
    plan = nb.nna_plan_trainable(made[kind]())
    gen = torch.Generator().manual_seed(B * L)
    x = torch.randn((B, L), generator=gen).cuda()
    run = {"stft": nb.nna_stft, "mel": lambda p, x: nb.nna_mel_with_stft(p, x)[0], "cqt": nb.nna_cqt}[kind]
    out, kept = nb.nna_forward_keep(plan, x)
    assert torch.equal(out, run(plan, x))
    gout = torch.randn(out.shape, generator=gen).cuda()
    gm, gw, gx = nb.nna_backward_kept(plan, x, gout, kept, want_gmelw=kind == "mel")
    want = {"stft": nb.nna_stft_backward, "mel": nb.nna_mel_backward, "cqt": nb.nna_cqt_backward}[kind](plan, x, gout)
    for got, ref in zip((gm, gw, gx), want if kind == "mel" else (None, *want)):
        _close(got, ref)
    with pytest.raises(nb.NnaError):
        nb.nna_backward_kept(plan, x, gout, kept[:-256])


@pytest.mark.parametrize("kind,hop,n_bins,B,L", [
    ("large", 32, 31, 200, 9001),     # 56,400 frames, above every line: cqt_kernel
    ("large", 96, 41, 260, 20003),    # ... its tiles across waveforms, a row block of one bin
    ("straight", 48, 31, 3, 5001),    # a hop that is no multiple of 32: the kernel that reads samples from memory
    ("straight", 8, 9, 5, 2051),
    ("respaced", 100, 131, 3, 7003), ("respaced", 100, 1, 1, 2100), ("respaced", 128, 200, 40, 9001)])
def test_other_kernels(kind, hop, n_bins, B, L):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] kept {kind} {hop} {n_bins} {B}x{L}", file=sys.stderr, flush=True)
    if kind == "respaced":
        plan = nb.nna_plan_stft_scaled(sr=16000, n_fft=400, hop=hop, freq_scale=nb.NNA_FREQ_LOG, fmin=60.0, fmax=6000.0, freq_bins=n_bins,
                                       fmt=nb.NNA_OUT_POWER, device=0)
        run, backward = nb.nna_stft, nb.nna_stft_backward
    else:
        plan = nb.nna_plan_cqt(sr=8000, hop=hop, fmin=80.0 if hop > 8 else 400.0, n_bins=n_bins, bins_per_octave=12, fmt=nb.NNA_OUT_LOG, device=0)
        run, backward = nb.nna_cqt, nb.nna_cqt_backward
    plan = nb.nna_plan_trainable(plan)
    gen = torch.Generator().manual_seed(B * L)
    x = torch.randn((B, L), generator=gen).cuda()
    out, kept = nb.nna_forward_keep(plan, x)
    assert torch.equal(out, run(plan, x))
    gout = torch.randn(out.shape, generator=gen).cuda()
    _, gw, gx = nb.nna_backward_kept(plan, x, gout, kept)
    for got, ref in zip((gw, gx), backward(plan, x, gout)):
        _close(got, ref)


def test_plans_that_keep_nothing():
    from paper_1912_12055_amd import binding as nb
    for plan in (nb.nna_plan_stft(fmt=nb.NNA_OUT_MAGNITUDE, device=0), nb.nna_plan_stft(fmt=nb.NNA_OUT_COMPLEX, device=0),
                 nb.nna_plan_mel(power=1.0, device=0), nb.nna_plan_cqt(fmin=220.0, n_bins=24, fmt=nb.NNA_OUT_COMPLEX, device=0)):
        assert nb.nna_kept_bytes(nb.nna_plan_trainable(plan), 2, 30000) == 0
    with pytest.raises(nb.NnaError):
        nb.nna_kept_bytes(nb.nna_plan_stft(device=0), 2, 30000)  # not trainable


@pytest.mark.parametrize("kind", ["stft", "mel", "cqt"])
def test_layers(kind, monkeypatch):
    import torch
    from paper_1912_12055_amd import layers
    made = {"stft": lambda: layers.STFT(n_fft=512, hop_length=128, output_format="Power", trainable=True),
            "mel": lambda: layers.MelSpectrogram(n_fft=512, hop_length=128, n_mels=40, trainable_mel=True, trainable_STFT=True),
            "cqt": lambda: layers.CQT1992v2(sr=8000, hop_length=32, fmin=80.0, n_bins=20, trainable=True)}
    layer = made[kind]()
    x = torch.randn((2, 5001), generator=torch.Generator().manual_seed(3)).cuda().requires_grad_()
    wanted = list(layer.parameters()) + [x]
    out = layer(x)
    gout = torch.randn(out.shape, generator=torch.Generator().manual_seed(4)).cuda()
    first = torch.autograd.grad(out, wanted, gout, retain_graph=True)
    again = torch.autograd.grad(out, wanted, gout)
    monkeypatch.setattr(layers, "_KEPT_BYTES", 0)  # every batch is too large
    out2 = layer(x)
    assert torch.equal(out, out2)
    for a, b, c in zip(first, again, torch.autograd.grad(out2, wanted, gout)):
        _close(a, c)
        _close(b, c)
    monkeypatch.undo()
    monkeypatch.setattr(layers.nb, "nna_forward_keep", None)  # without a backward pass to come nothing is kept
    with torch.no_grad():
        assert torch.equal(layer(x), out)


@pytest.mark.parametrize("kind", ["stft", "mel", "cqt"])
def test_bank_set_between_the_passes(kind):
    """A forward pass, new kernels, another forward pass, then the first one's backward pass: gradients with the new kernels throughout."""
    import torch
    from paper_1912_12055_amd import binding as nb, layers
    print(f"[case] kept bank {kind}", file=sys.stderr, flush=True)
    made = {"stft": lambda: layers.STFT(n_fft=512, hop_length=128, output_format="Power", trainable=True),
            "mel": lambda: layers.MelSpectrogram(n_fft=512, hop_length=128, n_mels=40, trainable_mel=True, trainable_STFT=True),
            "cqt": lambda: layers.CQT1992v2(sr=8000, hop_length=32, fmin=80.0, n_bins=20, trainable=True)}
    layer = made[kind]()
    bank = layer.cqt_kernels if kind == "cqt" else layer.wsin_wcos
    gen = torch.Generator().manual_seed(5)
    x = torch.randn((2, 5001), generator=gen).cuda().requires_grad_()
    out = layer(x)
    gout = torch.randn(out.shape, generator=gen).cuda()
    with torch.no_grad():
        bank.mul_(1.0 + 0.1 * torch.randn(bank.shape, generator=gen).cuda())
    layer(x[:1].detach())
    got = torch.autograd.grad(out, [bank, x], gout)
    backward = {"stft": nb.nna_stft_backward, "mel": nb.nna_mel_backward, "cqt": nb.nna_cqt_backward}[kind]
    for g, want in zip(got, backward(layer.plan, x.detach(), gout)[-2:]):
        _close(g, want)
