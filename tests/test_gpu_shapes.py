"""Default launch shapes on both sides of every size at which they change:
bit-exact framebuffers against the oracle."""
import pytest

from gpu_util import assert_same_fb, oracle_frame, read_fb, render_frame, upload
from paper_2104_07526_amd import pcr, synth

pytestmark = pytest.mark.gpu


def cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("variant", [pcr.BASIC, pcr.DEDUP, pcr.HQ, pcr.BASIC | pcr.F_LDS, pcr.HQ | pcr.F_PLAIN])
@pytest.mark.parametrize("per_cu", [2000, 3000, 5000])
def test_sizes_around_a_shape_change(orc, variant, per_cu):
    W, H = 320, 180
    pts = synth.terrain(per_cu * cus(), seed=7)
    m = synth.terrain_oblique(W, H)
    d = upload(pts)
    for n in (len(pts) - 1, len(pts)):
        efb, _ = oracle_frame(orc, pts[:n], m, W, H, variant)
        fb, _ = render_frame(d, m, W, H, variant, n=n)
        assert_same_fb(read_fb(fb, W, H, variant), efb, variant)


@pytest.mark.parametrize("size", [(320, 180), (1920, 1080)])     # above and below 8 points per pixel
def test_hq_large_tiles(orc, size):
    W, H = size
    pts = synth.terrain(40_000 * cus(), seed=8)
    m = synth.terrain_oblique(W, H)
    d = upload(pts)
    for n in (len(pts) - 1, len(pts)):
        efb, _ = oracle_frame(orc, pts[:n], m, W, H, pcr.HQ)
        fb, _ = render_frame(d, m, W, H, pcr.HQ, n=n)
        assert_same_fb(read_fb(fb, W, H, pcr.HQ), efb, pcr.HQ)
