"""The STFT layers' fast Fourier transform on batches large enough for its widest tiles and for several tiles per workgroup: frames
are independent of each other, so every waveform of a batch of repeated ones gets, bit for bit, what it gets alone."""
import sys

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    from paper_1912_12055_amd import binding
    binding.lib()
    return binding


def _repeated(seed, L, T, frames):
    import torch
    base = torch.randn((7, L), generator=torch.Generator().manual_seed(seed)).cuda()
    B = 7 * (-(-frames // (7 * T)))
    return base, base.repeat(B // 7, 1)


def _same(batch, alone):
    import torch
    out = batch.view(-1, 7, *alone.shape[1:])
    assert torch.isfinite(alone).all()
    assert torch.equal(out, alone[None].expand_as(out))


# a tile of 64 frames of 259 words: more than 64 KB of LDS, from 32,768 frames on
@pytest.mark.parametrize("fmt", ["COMPLEX", "PHASE"])
def test_complex_256(nb, fmt):
    print(f"[case] fft wide 256 {fmt}", file=sys.stderr, flush=True)
    base, x = _repeated(5, 3001, 1 + 3001 // 64, 33000)
    plan = nb.nna_plan_stft(n_fft=256, hop=64, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0)
    _same(nb.nna_stft(plan, x), nb.nna_stft(plan, base))


# n_fft, hop: frames beyond 1,024 steps of the kernel's frames per step (64 .. 2): several steps per tile, several tiles per workgroup,
# a ragged last tile; the general kernel past 1,024 tiles
SIZES = [(64, 16, 70001), (256, 64, 35001), (512, 160, 18001), (1024, 256, 9001), (2048, 441, 4601), (2048, 512, 9003), (4096, 1024, 2303), (4096, 512, 5001),
         (400, 160, 17001), (882, 441, 17001), (3000, 750, 9001), (12000, 3000, 1301)]


@pytest.mark.parametrize("n_fft,hop,frames", SIZES)
@pytest.mark.parametrize("fmt", ["MAGNITUDE", "LOG", "COMPLEX"])
def test_several_tiles_per_workgroup(nb, n_fft, hop, frames, fmt):
    print(f"[case] fft wide n_fft={n_fft} hop={hop} {fmt}", file=sys.stderr, flush=True)
    L = 11 * hop + n_fft // 2 + 3
    base, x = _repeated(n_fft + hop, L, 1 + L // hop, frames)
    plan = nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0)
    _same(nb.nna_stft(plan, x), nb.nna_stft(plan, base))


@pytest.mark.parametrize("n_fft,hop,frames", SIZES)
def test_mel_several_tiles_per_workgroup(nb, n_fft, hop, frames):
    print(f"[case] fft wide mel n_fft={n_fft} hop={hop}", file=sys.stderr, flush=True)
    L = 7 * hop + n_fft // 2 + 2
    base, x = _repeated(n_fft + hop + 1, L, 1 + L // hop, frames)
    plan = nb.nna_plan_mel(n_fft=n_fft, hop=hop, n_mels=40, device=0)
    alone = nb.nna_mel_with_stft(plan, base)
    for got, want in zip(nb.nna_mel_with_stft(plan, x), alone):
        _same(got, want)
    _same(nb.nna_mel(plan, x), alone[0])
