"""The constant-Q layers with frequency-domain kernels: both stages as one kernel bank (fixed kernels) against the oracle and
against the two-stage kernel (the same plan made trainable), at tile edges, every output format, one bin to 100."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
# the two-stage form rounds the spectrum and the spectral kernels to float32 on the way (relative 6e-8 each, sums of n_fft terms
# of random sign): 1e-6 .. 1e-5 of the peak measured for either form
TOL = 5e-5


@pytest.fixture(scope="module")
def nb():
    from paper_1912_12055_amd import binding
    binding.lib()
    return binding


def _wave(seed, B, L):
    rng = np.random.default_rng([23, seed])
    return (0.3 * rng.standard_normal((B, L))).astype(np.float32)


@pytest.mark.parametrize("fmt", ["MAGNITUDE", "POWER", "COMPLEX"])
@pytest.mark.parametrize("n_bins,bpo,hop,n_fft,B,L,center", [
    (1, 12, 64, 0, 1, 3000, True), (8, 12, 100, 0, 3, 2600, True), (9, 12, 16, 2048, 2, 4097, False),
    (36, 12, 128, 0, 7, 5000, True), (100, 24, 256, 0, 2, 9000, True)])
def test_composed_kernels(nb, fmt, n_bins, bpo, hop, n_fft, B, L, center):
    import torch
    cfg = dict(sr=8000, hop=hop, fmin=110.0, n_bins=min(n_bins, 5 * bpo), bins_per_octave=bpo, n_fft=n_fft)
    print(f"[case] composed {cfg} B={B} L={L} {fmt}", file=sys.stderr, flush=True)
    x = _wave(n_bins + hop, B, L)
    xd = torch.from_numpy(x).to("cuda:0")
    plan = nb.nna_plan_cqt1992(center=center, fmt=getattr(nb, "NNA_OUT_" + fmt), device=0, **cfg)
    got = nb.nna_cqt1992(plan, xd).cpu().numpy().astype(np.float64)
    two = nb.nna_cqt1992(nb.nna_plan_trainable(plan), xd).cpu().numpy().astype(np.float64)
    peak = np.abs(two).max()
    assert got.shape == two.shape and np.abs(got - two).max() < TOL * peak
    if fmt == "MAGNITUDE":
        ref = oracle.cqt1992(x, center=center, **cfg)
        assert np.abs(got - ref).max() < TOL * np.abs(ref).max()
