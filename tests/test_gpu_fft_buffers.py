"""The Fourier transform's tiles in two LDS buffers: frames do not depend on how many tiles their workgroup takes, nor on its number of
waves, so a waveform of a large batch gets, bit for bit, what it gets alone."""
import sys

import pytest

pytestmark = pytest.mark.gpu


# frames from one tile per workgroup to five and a remainder; waveforms shorter and longer than a tile
@pytest.mark.parametrize("frames", [4095, 4097, 12289, 20500])
@pytest.mark.parametrize("n_fft,hop,T", [(1024, 256, 5), (1024, 256, 331), (2048, 512, 3), (2048, 512, 67)])
@pytest.mark.parametrize("fmt", ["MAGNITUDE", "COMPLEX"])
def test_stft(n_fft, hop, T, frames, fmt):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fft buffers n_fft={n_fft} hop={hop} T={T} frames={frames} {fmt}", file=sys.stderr, flush=True)
    L = max((T - 1) * hop, n_fft // 2) + 7
    base = torch.randn((5, L), generator=torch.Generator().manual_seed(frames)).cuda()
    plan = nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0)
    alone = nb.nna_stft(plan, base)
    B = -(-frames // alone.shape[2])
    x = base.repeat(-(-B // 5), 1)[:B].contiguous()
    out = nb.nna_stft(plan, x)
    assert torch.equal(out, alone.repeat(-(-B // 5), 1, 1)[:B])


# the Mel tables in LDS (128 bands) and in memory (512 bands of n_fft 4,096 and more)
@pytest.mark.parametrize("n_fft,hop,n_mels", [(2048, 512, 128), (2048, 512, 512), (4096, 512, 512), (512, 128, 40)])
@pytest.mark.parametrize("frames", [2047, 9000, 26001])
def test_mel(n_fft, hop, n_mels, frames):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fft buffers mel n_fft={n_fft} n_mels={n_mels} frames={frames}", file=sys.stderr, flush=True)
    base = torch.randn((3, 11 * hop + n_fft // 2 + 5), generator=torch.Generator().manual_seed(frames)).cuda()
    plan = nb.nna_plan_mel(n_fft=n_fft, hop=hop, n_mels=n_mels, device=0)
    alone = nb.nna_mel(plan, base)
    B = -(-frames // alone.shape[2])
    out = nb.nna_mel(plan, base.repeat(-(-B // 3), 1)[:B].contiguous())
    assert torch.equal(out, alone.repeat(-(-B // 3), 1, 1)[:B])
