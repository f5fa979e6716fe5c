"""Constant-Q kernels tap by tap: the samples a tile reads of every hop are those its kernels reach, not the hop's; and the calls that are
left to the general kernel."""
import pytest


@pytest.fixture(scope="module")
def nb():
    from paper_1912_12055_amd import binding
    binding.lib()
    return binding


def _octave(nb, sr, hop, longest, n_bins, bpo):
    fmin = sr / longest / (2.0 ** (1.0 / bpo) - 1.0)
    plan = nb.nna_plan_part(nb.nna_plan_cqt2010v2(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, device=-1), 0)
    return plan, int(nb.nna_plan_cqt_lengths(plan)[0])


@pytest.mark.parametrize("hop,longest,n_bins,bpo", [(512, 120, 12, 12), (512, 250, 24, 24), (1024, 100, 12, 12), (1000, 350, 12, 12), (1500, 1400, 12, 12),
                                                    (4096, 1400, 24, 24), (2048, 70, 12, 12), (1024, 400, 36, 36)])
@pytest.mark.parametrize("frames", [300, 6000, 60000, 300000])
def test_kernels_shorter_than_a_hop(nb, hop, longest, n_bins, bpo, frames):
    plan, longest = _octave(nb, 44100, hop, longest, n_bins, bpo)
    form, tile, _, width = nb.nna_plan_short_tiles(plan, max(1, frames // 346), 345 * hop)
    # whole steps of 32, begun and ended on whole steps
    assert form >= 0 and tile >= 12 and longest <= width < longest + 62


@pytest.mark.parametrize("hop,longest,n_bins,bpo,width", [(512, 600, 12, 12, 512), (64, 700, 24, 24, 64), (1000, 1600, 12, 12, 1000),
                                                          (512, 486, 36, 36, 512), (12, 100, 12, 12, 12)])
def test_whole_hops(nb, hop, longest, n_bins, bpo, width):
    plan, _ = _octave(nb, 44100, hop, longest, n_bins, bpo)
    assert nb.nna_plan_short_tiles(plan, 3, 60 * hop)[3] == width


def test_tiles_of_few_frames_in_a_large_batch(nb):
    """Kernels of 1.6 hops of 1,000 samples, 36 bins: sixteen frames fill a CU's LDS; the general kernel takes 200,000 frames of them sooner."""
    plan, _ = _octave(nb, 44100, 1000, 1600, 36, 36)
    assert nb.nna_plan_short_tiles(plan, 17, 345 * 1000)[:2] == (2, 16)
    assert nb.nna_plan_short_tiles(plan, 578, 345 * 1000)[0] == -1
