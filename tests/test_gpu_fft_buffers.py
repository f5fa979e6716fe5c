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


# frames of two waves: one buffer of two steps or four (80 bands, tables in memory) where two buffers hold one step, one tile a workgroup
# and several, a last tile of any size (four steps: 12,203 frames)
@pytest.mark.parametrize("kind,n_mels", [("COMPLEX", 0), ("PHASE", 0), ("MAGNITUDE", 0), ("mel", 40), ("mel", 80), ("mel", 512)])
@pytest.mark.parametrize("frames", [1021, 1027, 2051, 4100, 9003, 12203])
def test_frames_of_two_waves(kind, n_mels, frames):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fft buffers 4096 {kind}{n_mels} frames={frames}", file=sys.stderr, flush=True)
    n_fft, hop = 4096, 512
    base = torch.randn((3, 16 * hop + 5), generator=torch.Generator().manual_seed(frames)).cuda()
    if kind == "mel":
        plan, run = nb.nna_plan_mel(n_fft=n_fft, hop=hop, n_mels=n_mels, device=0), nb.nna_mel
    else:
        plan, run = nb.nna_plan_stft(n_fft=n_fft, hop=hop, fmt=getattr(nb, "NNA_OUT_" + kind), device=0), nb.nna_stft
    alone = run(plan, base)
    B = -(-frames // alone.shape[2])
    out = run(plan, base.repeat(-(-B // 3), 1)[:B].contiguous())
    assert torch.equal(out, alone.repeat(-(-B // 3), 1, 1)[:B])
