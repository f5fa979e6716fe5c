"""The decimation filter of the downsampling constant-Q layers on the bfloat16 matrix pipe: lengths at the edges of its tiles (2,048 outputs,
256 a wave, 16 a column, rows that are not aligned), the longest and shortest filters that run there, samples that are not finite."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

KW = dict(sr=22050, hop=64, fmin=2000.0, n_bins=24, bins_per_octave=12)  # the lower octave reads the filter's output


@pytest.mark.parametrize("fir", [0, 131, 289])
@pytest.mark.parametrize("B,L", [(3, 513), (2, 767), (2, 4064), (1, 4095), (5, 4097), (2, 8192), (3, 8706), (700, 4100)])
def test_lengths(B, L, fir):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fir {fir} {B}x{L}", file=sys.stderr, flush=True)
    x = np.random.default_rng([7, L, fir]).standard_normal((B, L)).astype(np.float32)
    plan = nb.nna_plan_cqt2010v2(fir_taps=fir, fmt=nb.NNA_OUT_COMPLEX, device=0, **KW)
    got = nb.nna_cqt2010v2(plan, torch.from_numpy(x).cuda()).cpu().numpy()[-3:]
    ref = oracle.cqt2010v2(x[-3:], fir_taps=fir or oracle.FIR_TAPS, fmt=oracle.COMPLEX, **KW)
    low = slice(0, 24)
    # 130 products and 128 taps in float32, each sum off by less than sqrt(130) / 2 roundings of 6e-8: 1e-6 of the norm
    assert np.linalg.norm(got[:, low] - ref[:, low]) <= 1e-6 * np.linalg.norm(ref[:, low])


@pytest.mark.parametrize("scale", [2.0 ** -100, 2.0 ** 100])
def test_range(scale):
    """Samples as three bfloat16: nothing is lost from 2^-110 up (measured: 1.7e-7 from 1e-33 to 3e37, 2.6e-7 at 1e-34, 1.9e-5 at 1e-36)."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fir range {scale}", file=sys.stderr, flush=True)
    x = np.random.default_rng(7).standard_normal((2, 8706)).astype(np.float32)
    plan = nb.nna_plan_cqt2010v2(fmt=nb.NNA_OUT_COMPLEX, device=0, **KW)
    got = nb.nna_cqt2010v2(plan, torch.from_numpy(x * np.float32(scale)).cuda()).cpu().numpy()[:, :24].astype(np.float64) / scale
    ref = oracle.cqt2010v2(x, fmt=oracle.COMPLEX, **KW)[:, :24]
    assert np.linalg.norm(got - ref) <= 1e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3.4e38])
def test_reach_of_one_sample(bad):
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fir nonfinite {bad}", file=sys.stderr, flush=True)
    B, L, at, b = 3, 9001, 4097, 1
    x = np.random.default_rng(8).standard_normal((B, L)).astype(np.float32)
    x[b, at] = 0.0
    plan = nb.nna_plan_cqt2010v2(fmt=nb.NNA_OUT_COMPLEX, device=0, **KW)
    clean = nb.nna_cqt2010v2(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    x[b, at] = bad
    got = nb.nna_cqt2010v2(plan, torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.array_equal(np.delete(got, b, 0), np.delete(clean, b, 0))
    # a frame of the lower octave is 128 taps of every second sample about 64 t, each 128 samples either side through the filter
    t = 64 * np.arange(got.shape[2])
    clear = np.abs(t - at) > 2 * 64 + 128 + 2
    assert np.abs(got[b][:24, clear] - clean[b][:24, clear]).max() <= 1e-5 * np.abs(clean[b][:24]).max()
    if not np.isfinite(bad):
        assert not np.isfinite(got[b][:24, np.abs(t - at) < 64]).any()


@pytest.mark.parametrize("fir", [131, 255, 257])
def test_reach_is_the_filters_own_taps(fir):
    """Outputs of the filter that none of its taps reach a NaN from: seen through the lower octave's kernels, whose steps of sixteen taps
    begin at every 32nd output, for a NaN on each of 32 consecutive odd samples."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print(f"[case] fir reach {fir}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt2010v2(fir_taps=fir, fmt=nb.NNA_OUT_COMPLEX, device=0, **KW)
    top = nb.nna_plan_part(plan, 0)
    lengths, half = nb.nna_plan_cqt_lengths(top), top.info()["taps"] // 2
    B, L = 32, 9001
    x = np.tile(np.random.default_rng(9).standard_normal(L).astype(np.float32), (B, 1))
    at = 4097 + 2 * np.arange(B)
    x[np.arange(B), at] = np.nan
    got = np.isfinite(nb.nna_cqt2010v2(plan, torch.from_numpy(x).cuda()).cpu().numpy())[:, :24].reshape(B, 12, 2, -1)
    y = np.arange(L // 2 + 1)
    reached = np.abs(2 * y[None] - at[:, None]) <= fir // 2  # (an odd offset: never a tap that is zero)
    for block in (slice(0, 8), slice(8, 12)):  # bins whose kernels share their steps
        n = int(lengths[block].max())
        lo, hi = (half - (n + 1) // 2) // 16 * 16, (half + n // 2 + 15) // 16 * 16
        for t in range(got.shape[3]):
            window = slice(max(0, 32 * t - half + lo), max(0, 32 * t - half + hi))
            clear = ~reached[:, window].any(1)
            assert got[clear, block, :, t].all(), (fir, t, at[clear][~got[clear, block, :, t].all((1, 2))])


def test_cost_of_samples_that_are_not_finite():
    """A recording full of them, or with one in every frame, keeps to a small multiple of the time of one without."""
    import torch
    from paper_1912_12055_amd import binding as nb
    print("[case] fir nonfinite cost", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt2010v2(fmt=nb.NNA_OUT_COMPLEX, device=0, **KW)
    clean = torch.randn((400, 100000), generator=torch.Generator().manual_seed(1)).cuda()
    some = clean.clone()
    some[:, 137::1000] = float("nan")

    def milliseconds(x):
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            nb.nna_cqt2010v2(plan, x)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    base = milliseconds(clean)  # (tap by tap from memory: 28 and 15 times as long)
    assert milliseconds(torch.full_like(clean, float("nan"))) < 7 * base
    assert milliseconds(some) < 7 * base
