"""Where the constant-Q calls of the binding take their workspace from, without a GPU: torch's streams and allocator and the library's calls
are stand-ins that record what is asked of them."""
import contextlib
import ctypes

import pytest
import torch

from paper_1912_12055_amd import binding as nb

NEED = 4096


class _Memory:
    def __init__(self, owner):
        self.owner = owner

    def data_ptr(self):
        return 1 << 20


@pytest.fixture
def calls(monkeypatch):
    """Of every call [entry point, stream it ran on, stream its memory was taken on]; `current` is torch's current stream."""
    seen = dict(calls=[], current=0x700, taken=None, kind=nb.NNA_KIND_CQT)

    class Library:
        @staticmethod
        def entry(name):
            def call(handle, xp, B, L, op, *rest):
                seen["calls"].append((name, rest[-1], seen["taken"] if len(rest) == 3 else None))
                return nb.NNA_OK
            return call

    library = Library()
    for name in ("nna_cqt", "nna_cqt1992", "nna_cqt_in_workspace"):
        setattr(library, name, Library.entry(name))

    def run(fn, plan, x, out, stream):
        return fn(plan.handle, 0, 2, 100, 0, seen["current"] if stream is None else stream)

    class ExternalStream:
        pool = 0x1000

        def __init__(self, stream_ptr, device=None):
            if not isinstance(stream_ptr, int):
                raise TypeError("an integer is required")
            # as torch's: no handle given, the next stream of the pool
            type(self).pool += 16
            self.cuda_stream = stream_ptr or type(self).pool

    class DefaultStream:
        cuda_stream = 0

    @contextlib.contextmanager
    def on(stream):
        before, seen["current"] = seen["current"], stream.cuda_stream
        yield
        seen["current"] = before

    def empty(n, dtype=None, device=None):
        assert n == NEED
        seen["taken"] = seen["current"]
        return _Memory(seen["current"])

    class Plan:
        handle = 1

        def constants(self):
            return seen["kind"], 0, 0

    class X:
        device = torch.device("cuda:0")

    monkeypatch.setattr(nb, "lib", lambda: library)
    monkeypatch.setattr(nb, "_run", run)
    monkeypatch.setattr(nb, "nna_cqt_workspace", lambda plan, B, L: NEED)
    monkeypatch.setattr(torch.cuda, "ExternalStream", ExternalStream)
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: DefaultStream())
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: type("Current", (), dict(cuda_stream=seen["current"])))
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    seen["plan"], seen["x"] = Plan(), X()
    return seen


# no stream given, the default stream's handle, a stream of the program's
@pytest.mark.parametrize("stream", [None, 0, 0x5550])
def test_memory_is_of_the_stream_the_call_runs_on(calls, stream):
    nb.nna_cqt(calls["plan"], calls["x"], stream=stream)
    (name, ran, taken), = calls["calls"]
    assert name == "nna_cqt_in_workspace"
    assert ran == taken == (0x700 if stream is None else stream)


# HIP's handles for "the default stream" and "this thread's stream" are no streams of torch's; a handle that is not a number
@pytest.mark.parametrize("stream", [1, 2, ctypes.c_void_p(0x5550)], ids=str)
def test_handles_that_name_no_one_stream_take_no_memory(calls, stream):
    nb.nna_cqt(calls["plan"], calls["x"], stream=stream)
    assert calls["calls"] == [("nna_cqt", stream, None)]


def test_no_memory_left(calls, monkeypatch):
    def empty(*a, **k):
        raise torch.OutOfMemoryError("none")
    monkeypatch.setattr(torch, "empty", empty)
    nb.nna_cqt(calls["plan"], calls["x"])
    assert calls["calls"] == [("nna_cqt", 0x700, None)]


def test_a_plan_of_the_other_kind_goes_to_the_entry_point_that_refuses_it(calls):
    for kind, call in ((nb.NNA_KIND_CQT1992, nb.nna_cqt), (nb.NNA_KIND_CQT, nb.nna_cqt1992)):
        calls["kind"] = kind
        call(calls["plan"], calls["x"])
    assert [c[0] for c in calls["calls"]] == ["nna_cqt", "nna_cqt1992"]


# a graph that torch captures has a pool of its own, one captured by other means has not
@pytest.mark.parametrize("pool,name", [((0, 3), "nna_cqt_in_workspace"), ((0, 0), "nna_cqt")])
@pytest.mark.parametrize("stream", [None, 0x5550])
def test_under_capture(calls, monkeypatch, stream, pool, name):
    segments = [dict(address=1 << 12, total_size=1 << 12, segment_pool_id=(0, 9)), dict(address=1 << 19, total_size=1 << 20, segment_pool_id=pool)]
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    monkeypatch.setattr(torch.cuda, "memory_snapshot", lambda: segments)
    nb.nna_cqt(calls["plan"], calls["x"], stream=stream)
    assert [c[0] for c in calls["calls"]] == [name]


def test_current_stream_of_another_device(calls, monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 1)
    nb.nna_cqt(calls["plan"], calls["x"])
    assert calls["calls"] == [("nna_cqt_in_workspace", 0x700, 0x700)]
