"""Constant-Q calls whose hop-blocks' coordinates go through the caller's memory, against the one launch that keeps them in LDS: every
width of tile and kind of item beside them, waveforms in parts, hops that are no multiple of 64, samples that are not finite."""
import sys

import numpy as np
import pytest

from test_gpu_hopblocks import CASES, nb  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu
# the same coordinates, products and blocks of 32 products; up to 108 block sums added in another order: 108 x 2^-24 of a bin's own sums at
# most, 4e-7 of the peak measured
TOL = 2e-6


def _one_launch(nb, plan, x):
    return nb._run(nb.lib().nna_cqt1992 if plan.info()["kind"] == nb.NNA_KIND_CQT1992 else nb.lib().nna_cqt, plan, x, None, None)


def _both(nb, plan, x, floats):
    import torch
    ws = torch.full((floats,), float("nan"), device="cuda:0")
    return nb.nna_cqt_in_workspace(plan, x, ws).cpu().numpy(), _one_launch(nb, plan, x).cpu().numpy()


def _written(ws):
    """Words of a workspace that was all NaN up to the last one that a call wrote."""
    at = (~ws.isnan()).nonzero()
    return int(at[-1]) + 1 if len(at) else 0


def _floats_of_a_waveform(nb, plan, x):
    import torch
    ws = torch.full((1 << 24,), float("nan"), device="cuda:0")
    nb.nna_cqt_in_workspace(plan, x[:1], ws)
    assert 0 < _written(ws) < len(ws)
    return _written(ws)


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[3]}-{c[6]}x{c[7]}")
def test_against_one_launch(nb, case):
    import torch
    n_bins, bpo, sr, hop, fmin, n_taps, B, L, center, tiles = case
    print(f"[case] cqt workspace {case}", file=sys.stderr, flush=True)
    x = torch.from_numpy((0.3 * np.random.default_rng([31, n_bins, hop]).standard_normal((B, L))).astype(np.float32)).to("cuda:0")
    for fmt in (nb.NNA_OUT_MAGNITUDE, nb.NNA_OUT_COMPLEX):
        plan = nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, n_taps=n_taps, center=center, fmt=fmt, device=0)
        got, ref = _both(nb, plan, x, 1 << 24)
        assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
        for share in {B // 3, 2 * B // 3} - {0}:  # in parts of unequal size where B is no multiple of them
            parts = -(-B // share)
            each = _floats_of_a_waveform(nb, plan, x)
            assert share < B and parts > 1
            ws = torch.full((share * each,), float("nan"), device="cuda:0")
            got = nb.nna_cqt_in_workspace(plan, x, ws).cpu().numpy()
            assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
            # the coordinates of the largest part, every word of them, and no more
            assert _written(ws) == -(-B // parts) * each and not ws[:-(-B // parts) * each].isnan().any()
        got, ref = _both(nb, plan, x, 16)  # not one waveform's: not used
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("B,L,n_bins,hop", [(1, 16390, 84, 512), (3, 40001, 84, 512), (70, 9000, 60, 256)])
def test_dense_kernels(nb, B, L, n_bins, hop):
    import torch
    print(f"[case] cqt workspace dense {B} {L} {n_bins} {hop}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt1992(sr=22050, hop=hop, n_bins=n_bins, fmin=32.7 if n_bins == 84 else 65.4, fmt=nb.NNA_OUT_COMPLEX, device=0)
    x = torch.from_numpy((0.3 * np.random.default_rng([33, B]).standard_normal((B, L))).astype(np.float32)).to("cuda:0")
    assert nb.nna_cqt_workspace(plan, B, L) > 0
    got, ref = _both(nb, plan, x, nb.nna_cqt_workspace(plan, B, L) // 4)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
    assert np.array_equal(nb.nna_cqt1992(plan, x).cpu().numpy(), got)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3.3e38])
def test_not_finite(nb, bad):
    """The outputs that a bad sample reaches, and no others, whichever way the coordinates go."""
    import torch
    print(f"[case] cqt workspace {bad}", file=sys.stderr, flush=True)
    x = torch.from_numpy((0.3 * np.random.default_rng(35).standard_normal((3, 60001))).astype(np.float32)).to("cuda:0")
    x[1, 30011] = bad
    for plan in (nb.nna_plan_cqt(n_bins=84, fmt=nb.NNA_OUT_COMPLEX, device=0), nb.nna_plan_cqt1992(n_bins=84, fmt=nb.NNA_OUT_COMPLEX, device=0)):
        got, ref = _both(nb, plan, x, 1 << 24)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
        fine = np.isfinite(ref) & (np.abs(ref) < 1e10)
        assert fine.any() and np.abs(got - ref)[fine].max() <= TOL * np.abs(ref[fine]).max()


def test_memory_that_cannot_serve(nb):
    import torch
    plan = nb.nna_plan_cqt(n_bins=84, device=0)
    x = torch.randn((2, 40000), generator=torch.Generator().manual_seed(1)).cuda()
    ref = _one_launch(nb, plan, x)
    ws = torch.empty(1 << 22, device="cuda:0")
    assert torch.equal(nb.nna_cqt_in_workspace(plan, x, ws[1:]), ref)  # not aligned to 16 bytes
    kept = nb.nna_plan_trainable(plan)  # trained kernels are contracted
    assert nb.nna_cqt_workspace(kept, 2, 40000) == 0
    assert torch.equal(nb.nna_cqt_in_workspace(kept, x, ws), _one_launch(nb, kept, x))
    with pytest.raises(RuntimeError):
        nb.nna_cqt_workspace(nb.nna_plan_stft(n_fft=256, hop=64, device=0), 2, 4000)
    with pytest.raises(RuntimeError):
        nb.nna_cqt_workspace(plan, 2, 100)


def test_memory_of_the_calls_stream(nb):
    """No stream, the default stream's handle, a side stream's: the same outputs, and the same memory call after call."""
    import torch
    x = torch.randn((4, 60001), generator=torch.Generator().manual_seed(2)).cuda()
    side = torch.cuda.Stream()
    for make, call in ((nb.nna_plan_cqt, nb.nna_cqt), (nb.nna_plan_cqt1992, nb.nna_cqt1992)):
        plan = make(sr=44100, n_bins=168, bins_per_octave=24, device=0) if call is nb.nna_cqt else make(n_bins=84, device=0)
        xs = x if nb.nna_cqt_workspace(plan, *x.shape) else torch.randn((20, 176400), generator=torch.Generator().manual_seed(3)).cuda()
        assert nb.nna_cqt_workspace(plan, *xs.shape) > 0
        print(f"[case] cqt memory by stream {call.__name__} {tuple(xs.shape)}", file=sys.stderr, flush=True)
        ref = call(plan, xs)
        out = torch.empty_like(ref)
        torch.cuda.synchronize()
        for stream in (0, side.cuda_stream):
            reserved = []
            for _ in range(40):  # (more than torch's pool has streams)
                out.fill_(float("nan"))
                torch.cuda.current_stream().synchronize()
                call(plan, xs, out=out, stream=stream)
                torch.cuda.synchronize()
                assert torch.equal(out, ref)
                reserved.append(torch.cuda.memory_reserved())
            assert len(set(reserved)) == 1, stream


def test_plans_of_the_other_kind_are_refused(nb):
    import torch
    x = torch.randn((16, 60001), generator=torch.Generator().manual_seed(4)).cuda()
    for plan, call in ((nb.nna_plan_cqt1992(n_bins=84, device=0), nb.nna_cqt), (nb.nna_plan_cqt(sr=44100, n_bins=168, bins_per_octave=24, device=0), nb.nna_cqt1992)):
        with pytest.raises(nb.NnaError) as e:
            call(plan, x)
        assert e.value.status == nb.NNA_ERR_INVALID_ARG


@pytest.mark.parametrize("by_torch", [True, False])
def test_replays(nb, by_torch):
    """A call in a graph, captured through torch or past it, replayed between eager work that takes and fills memory on every stream of the call."""
    import ctypes

    import torch
    print(f"[case] cqt memory in a graph {by_torch}", file=sys.stderr, flush=True)
    plan = nb.nna_plan_cqt1992(n_bins=84, device=0)
    x = torch.randn((2, 60001), generator=torch.Generator().manual_seed(5)).cuda()
    need = nb.nna_cqt_workspace(plan, *x.shape)
    assert need > 0
    out = nb.nna_cqt1992(plan, x)
    side = torch.cuda.Stream()
    nb.nna_cqt1992(plan, x, out=out, stream=side.cuda_stream)
    torch.cuda.synchronize()
    if by_torch:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            nb.nna_cqt1992(plan, x, out=out)
        replay = graph.replay
    else:
        hip, handle = nb.lib(), ctypes.c_void_p(side.cuda_stream)  # (the library brings HIP's runtime along)
        graph, run = ctypes.c_void_p(), ctypes.c_void_p()
        assert hip.hipStreamBeginCapture(handle, 2) == 0
        nb.nna_cqt1992(plan, x, out=out, stream=side.cuda_stream)
        assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
        assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0

        def replay():
            assert hip.hipGraphLaunch(run, handle) == 0
    for rep in range(3):
        x.copy_(torch.randn(x.shape, generator=torch.Generator().manual_seed(6 + rep)))
        for stream in (torch.cuda.current_stream(), side):
            with torch.cuda.stream(stream):
                taken = [torch.full((need // 4,), float("nan"), device="cuda:0") for _ in range(4)]
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        replay()
        torch.cuda.synchronize()
        # (a graph captured past torch runs in one launch, whose sums are added in another order)
        ref = nb.nna_cqt1992(plan, x) if by_torch else _one_launch(nb, plan, x)
        assert torch.equal(out, ref), rep
        assert all(bool(t.isnan().all()) for t in taken)
        del taken
    if not by_torch:
        assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0


# calls where two launches took 0.60 .. 0.94 of one's time, and where they took 1.06 .. 1.45
@pytest.mark.parametrize("sr,hop,fmin,n_bins,bpo,B,L,two", [
    (44100, 512, 32.7, 168, 24, 1770, 176400, True), (44100, 256, 32.7, 216, 36, 4, 225000, True), (22050, 1024, 32.7, 119, 24, 304, 1048000, True),
    (44100, 512, 32.7, 120, 24, 1, 794193, False), (22050, 256, 27.5, 119, 24, 1, 197033, False), (44100, 512, 32.7, 287, 36, 1, 249585, False),
    (44100, 512, 32.7, 84, 12, 122, 512000, False), (22050, 1024, 32.7, 67, 12, 461, 245013, False), (44100, 256, 27.5, 59, 12, 656, 37448, False)])
def test_two_launches_where_they_pay(nb, sr, hop, fmin, n_bins, bpo, B, L, two):
    plan = nb.nna_plan_cqt(sr=sr, hop=hop, fmin=fmin, n_bins=n_bins, bins_per_octave=bpo, device=0)
    assert (nb.nna_cqt_workspace(plan, B, L) > 0) == two


# a batch that the tiles take, in parts that they don't, and in parts short enough that they do again
@pytest.mark.parametrize("share,in_parts", [(40, False), (16, True)])
def test_parts_too_short_for_the_tiles(nb, share, in_parts):
    import torch
    plan = nb.nna_plan_cqt(sr=8000, hop=64, fmin=56.0, n_bins=60, bins_per_octave=24, device=0)
    B, L = 80, 32768
    print(f"[case] cqt workspace parts of {share}", file=sys.stderr, flush=True)
    assert nb.nna_plan_applied_tiles(plan, B, L)[0][0] and bool(nb.nna_plan_applied_tiles(plan, share, L)[0][0]) == in_parts
    x = torch.randn((B, L), generator=torch.Generator().manual_seed(9)).cuda()
    each = _floats_of_a_waveform(nb, plan, x)
    ws = torch.full((share * each,), float("nan"), device="cuda:0")
    got, ref = nb.nna_cqt_in_workspace(plan, x, ws), _one_launch(nb, plan, x)
    if in_parts:
        assert _written(ws) == share * each and (got - ref).abs().max() <= TOL * ref.abs().max()
    else:  # one launch, without the workspace
        assert _written(ws) == 0 and torch.equal(got, ref)
