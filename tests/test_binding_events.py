"""Events kept by a handle, on the CPU with stand-ins for torch's streams and
events: a call under another current device than the one before must not record
the event that belongs to the first device (torch refuses it), and calls under
one device must not create new ones."""
import pytest
import torch

from paper_1303_2470_amd import lbmp


class Event:
    made = 0

    def __init__(self):
        Event.made += 1
        self.device = None


class Stream:
    def __init__(self, device_index):
        self.device_index = device_index
        self.cuda_stream = 0
        self.waited = []

    def record_event(self, event=None):
        event = Event() if event is None else event
        if event.device not in (None, self.device_index):
            raise RuntimeError("Event device does not match recording stream's device")
        event.device = self.device_index
        return event

    def wait_event(self, event):
        self.waited.append(event)


@pytest.fixture()
def current(monkeypatch):
    state = {"stream": Stream(0)}
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: state["stream"])
    Event.made = 0
    return state


class Lib:
    """Accepts every call; no stream is idle."""

    def __getattr__(self, name):
        return lambda *a: 0


def test_current_device_changes_between_calls(current, monkeypatch):
    monkeypatch.setattr(lbmp, "_lib", Lib())
    mp = lbmp.MP(None, None, [], [1], Stream(0), None)
    streams = [Stream(0), Stream(1), Stream(0), Stream(1)]
    for s in streams:
        current["stream"] = s
        lbmp.mp_step_n(mp, 1)
    assert [e.device for e in mp.stream.waited] == [0, 1, 0, 1]
    made = Event.made
    for s in streams:
        current["stream"] = s
        lbmp.mp_step_n(mp, 1)
    assert Event.made == made == 2
