"""Which stream of an EPBuffer waits for what, with streams that only record it: no GPU."""
import contextlib
import threading

import pytest
import torch

from paper_2603_13606_amd import buffer


class Stream:
    def __init__(self, address):
        self.cuda_stream, self.waited, self.capturing = address, [], False

    def wait_event(self, event):
        if self.capturing:
            raise RuntimeError("a stream under graph capture can't wait for work outside the graph")
        self.waited.append(event)


@pytest.fixture
def buf(monkeypatch):
    """A buffer that has made one call, on the compute stream, and not yet given its communication stream away."""
    b = buffer.EPBuffer.__new__(buffer.EPBuffer)
    b.compute, b._comm, b._lock, b._comm_given = Stream(1), Stream(2), threading.Lock(), False
    b._order_event, b._order_streams = "first call", (1,)
    current = [b.compute]

    @contextlib.contextmanager
    def on(stream):
        current.append(stream)
        yield
        current.pop()

    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: current[-1].capturing)
    return b


def test_the_communication_stream_comes_behind_the_calls_made(buf):
    assert buf.get_comm_stream() is buf._comm and buf.comm_stream is buf._comm
    assert buf._comm.waited == ["first call"] and buf._comm_given


@pytest.mark.parametrize("drawn_in", [False, True])
def test_the_communication_stream_asked_for_under_capture_waits_later(buf, drawn_in):
    buf.compute.capturing, buf._comm.capturing = True, drawn_in
    assert buf.get_comm_stream() is buf._comm
    assert buf._comm.waited == [] and buf._comm_given
    buf.compute.capturing = buf._comm.capturing = False
    buf.get_comm_stream()
    assert buf._comm.waited == ["first call"]


def test_a_wait_that_fails_is_not_taken_for_done(buf, monkeypatch):
    with monkeypatch.context() as m:
        m.setattr(buf._comm, "wait_event", lambda e: 1 / 0)
        with pytest.raises(ZeroDivisionError):
            buf.get_comm_stream()
        assert not buf._comm_given
    buf.get_comm_stream()
    assert buf._comm.waited == ["first call"]


def test_another_communication_stream_can_be_set(buf):
    """It takes the calls from then on, behind the last one made."""
    other = Stream(3)
    buf.comm_stream = other
    assert buf.comm_stream is other and buf.get_comm_stream() is other and buf._comm_given
    assert other.waited == ["first call"]
