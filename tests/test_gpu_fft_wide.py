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
