"""Scattered tiles pass the LDS table by in frames of 1.6M visible points and
more; images below 196,608 pixels also ask for a visible share of 3/8.  Both
sides of these lines, with scattered, ordered and partly visible tiles in one
launch: bit-exact framebuffers against the oracle."""
import pytest

from gpu_util import assert_same_fb, oracle_frame, read_fb, render_frame, upload
from paper_2104_07526_amd import pcr
from test_gpu_scatter import mixed_cloud

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
@pytest.mark.parametrize("size", [(160, 120), (512, 383), (512, 384), (31, 7000)])
@pytest.mark.parametrize("n", [1_599_999, 1_600_001, 2_400_077, 4_000_001])
def test_both_sides_of_the_line(orc, variant, size, n):
    W, H = size
    pts, m = mixed_cloud(n, seed=n)
    efb, _ = oracle_frame(orc, pts, m, W, H, variant)
    d = upload(pts)
    for tune in (None, {"ppt": 1}, {"ppt": 2, "wg": 256}, {"ppt": 8, "grid": 500}, {"ppt": 16}):
        fb, _ = render_frame(d, m, W, H, variant, tune=tune)
        assert_same_fb(read_fb(fb, W, H, variant), efb, variant)


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
def test_chunks_and_views(orc, variant):
    """The same in a chunk table and in a batch's single-view passes."""
    import torch
    W, H = 640, 360
    n = 3_000_017
    pts, m = mixed_cloud(n, seed=5)
    efb, _ = oracle_frame(orc, pts, m, W, H, variant)
    d = upload(pts)
    ends = [0, 1, 700, 5000, 1_000_001, 2_999_000, n]
    tab = pcr.chunk_table([(d.data_ptr() + 16 * a, b - a) for a, b in zip(ends, ends[1:])])
    fb = pcr.alloc_fb(W, H, variant)
    pcr.fb_clear(fb, W, H, variant)
    pcr.render_chunks(tab, len(ends) - 1, m, W, H, variant, fb)
    assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
    kind = pcr.HQ if variant == pcr.HQ else pcr.BASIC
    image = torch.empty(W * H, dtype=torch.int32, device=d.device)
    plan = pcr.BatchPlan(d, 1, tune={"group": 1})
    plan.launch([pcr.make_view(m, W, H, kind, fb, image)])
    torch.cuda.synchronize()
    assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
    plan.close()
