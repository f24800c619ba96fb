"""The Python binding keeps the buffers that a batch launch writes alive: a
view record holds its framebuffer and image tensors, and launches hold them
until the event recorded after the launch has completed (CPU only: tensors on
the host, a stand-in event)."""
import gc
import weakref

import numpy as np
import pytest
import torch

from paper_2104_07526_amd import pcr


def test_view_record_holds_its_buffers():
    W, H = 8, 4
    fb = torch.empty(pcr.fb_bytes(W, H, pcr.BASIC) // 8, dtype=torch.int64)
    img = torch.empty(W * H, dtype=torch.int32)
    rf, ri = weakref.ref(fb), weakref.ref(img)
    v = pcr.make_view(np.eye(4), W, H, pcr.BASIC, fb, img)
    del fb, img
    gc.collect()
    assert rf() is not None and ri() is not None
    assert v.fb == rf().data_ptr() and v.rgba_out == ri().data_ptr()
    del v
    gc.collect()
    assert rf() is None and ri() is None


class FakeEvent:
    def __init__(self):
        self.done = False

    def query(self):
        return self.done


def test_launch_holds_buffers_until_completion():
    W, H = 8, 4
    held = pcr._InFlight()
    fb = torch.empty(pcr.fb_bytes(W, H, pcr.HQ) // 8, dtype=torch.int64)
    img = torch.empty(W * H, dtype=torch.int32)
    rf = weakref.ref(fb)
    views = [pcr.make_view(np.eye(4), W, H, pcr.HQ, fb, img)]
    ev = FakeEvent()
    held.hold(ev, pcr._held_refs(None, views))
    del fb, img, views
    gc.collect()
    assert rf() is not None and held.pending() == 1     # launch not complete: still held
    ev.done = True
    assert held.pending() == 0                          # completed: released
    gc.collect()
    assert rf() is None


def test_framebuffer_size_follows_a_size_that_changes():
    """Sizes may be 0-d arrays or tensors; one that changes in place gives the
    size of its present value, so a framebuffer that became too small is refused."""
    for one in (torch.tensor(64), np.array(64), np.int64(64)):
        pcr._fb_fits(torch.empty(64 * 64, dtype=torch.int64), one, 64, pcr.BASIC)
    fb, w = torch.empty(64 * 64, dtype=torch.int64), torch.tensor(64)
    pcr._fb_fits(fb, w, 64, pcr.BASIC)
    w.fill_(65)
    with pytest.raises(ValueError):
        pcr._fb_fits(fb, w, 64, pcr.BASIC)
    h, variant = torch.tensor(64), torch.tensor(pcr.BASIC)
    pcr._fb_fits(fb, 64, h, variant)
    variant.fill_(pcr.HQ)
    with pytest.raises(ValueError):
        pcr._fb_fits(fb, 64, h, variant)


@pytest.mark.parametrize("gone", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_of_a_torch_without_the_private_calls(monkeypatch, gone):
    class Stream:
        cuda_stream = 123

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.setattr(torch._C, name, lambda *a: 0, raising=False)
    monkeypatch.delattr(torch._C, gone)
    assert pcr._stream(None) == 123
