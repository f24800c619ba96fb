"""Default launch shapes on both sides of the lines that depend on the number of
points and on the image: bit-exact framebuffers against the oracle."""
import pytest

from gpu_util import assert_same_fb, oracle_frame, read_fb, render_frame, upload
from paper_2104_07526_amd import pcr, synth

pytestmark = pytest.mark.gpu


def cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


# points per compute unit and pixels per point at a line, image width
LINES = [(400, 3, 640), (1400, 8, 1920), (1400, 10 / 7, 640), (1400, 30 / 7, 640), (4000, 10 / 7, 640), (4000, 30 / 7, 1280),
         (4000, 1 / 3, 640)]


@pytest.mark.parametrize("variant", [pcr.BASIC, pcr.BASIC | pcr.F_EARLYZ, pcr.DEDUP, pcr.DEDUP | pcr.F_PLAIN,
                                     pcr.DEDUP | pcr.F_LDS, pcr.HQ, pcr.HQ | pcr.F_EARLYZ])
@pytest.mark.parametrize("per_cu,pixels,w", LINES)
def test_both_sides(orc, variant, per_cu, pixels, w):
    n = per_cu * cus()
    pts = synth.terrain(n, seed=7)
    d = upload(pts)
    for h in (int(pixels * n) // w, int(pixels * n) // w + 1):
        m = synth.terrain_oblique(w, h)
        for k in (n - 1, n):
            efb, _ = oracle_frame(orc, pts[:k], m, w, h, variant)
            fb, _ = render_frame(d, m, w, h, variant, n=k)
            assert_same_fb(read_fb(fb, w, h, variant), efb, variant)


@pytest.mark.parametrize("per_cu,pixels,w", [(1400, 30 / 7, 640), (4000, 30 / 7, 1280)])
def test_robust_sums(orc, per_cu, pixels, w):
    """The robust sums, whose image is the two-word one's."""
    n = per_cu * cus()
    pts = synth.terrain(n, seed=9)
    d = upload(pts)
    for h in (int(pixels * n) // w, int(pixels * n) // w + 1):
        m = synth.terrain_oblique(w, h)
        for k in (n - 1, n):
            _, eimg = oracle_frame(orc, pts[:k], m, w, h, pcr.HQ)
            _, img = render_frame(d, m, w, h, pcr.HQ | pcr.F_HQ_ROBUST, n=k)
            assert (img == eimg).all()
