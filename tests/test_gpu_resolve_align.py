"""Closest-point resolves into images that are only 4-byte aligned (one pixel a
thread) and 8-byte aligned (two pixels a thread): the same words, and nothing
written outside the image."""
import numpy as np
import pytest

from gpu_util import upload
from paper_2104_07526_amd import pcr, synth

pytestmark = pytest.mark.gpu

GUARD = 0x5A5A5A5A


@pytest.mark.parametrize("w,h", [(1, 1), (2, 1), (3, 1), (1, 2), (15, 17), (16, 16), (511, 1), (33, 31), (640, 361), (5_001, 1_677)])
@pytest.mark.parametrize("off", [2, 3, 4, 5])
def test_image_alignment(orc, w, h, off):
    import torch
    pts = synth.sphere(20_000, seed=4)
    m = synth.sphere_view(w, h)
    fb = pcr.alloc_fb(w, h, pcr.BASIC)
    pcr.fb_clear(fb, w, h, pcr.BASIC)
    pcr.render(upload(pts), m, w, h, pcr.BASIC, fb)
    room = torch.full((w * h + 8,), GUARD, dtype=torch.int32, device=fb.device)
    image = room[off:off + w * h]
    assert image.data_ptr() % 8 == 4 * (off % 2)
    pcr.resolve(fb, w, h, pcr.BASIC, out=image)
    torch.cuda.synchronize()
    got = room.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[off:off + w * h], orc.resolve_basic(orc.render_basic(pts, m, w, h), w, h))
    assert (got[:off] == GUARD).all() and (got[off + w * h:] == GUARD).all()
