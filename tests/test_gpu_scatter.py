"""Tiles whose points scatter over the image (unordered clouds) skip the LDS
table: bit-exact framebuffers with scattered, ordered and mixed tiles in one
launch, at every tile shape, against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same_fb, oracle_frame, read_fb, render_frame, upload
from paper_2104_07526_amd import pcr, synth

pytestmark = pytest.mark.gpu

W, H = 160, 120


def mixed_cloud(n, seed):
    """Blocks of 37 to 900 points in turn: random over the whole image, along a
    scanline, all on a few pixels, and outside the view."""
    rng = np.random.default_rng(seed)
    u, v = np.empty(n), np.empty(n)
    s, kind = 0, 0
    while s < n:
        e = min(n, s + int(rng.integers(37, 900)))
        k = e - s
        if kind == 0:
            u[s:e], v[s:e] = rng.uniform(-1, 1, k), rng.uniform(-1, 1, k)
        elif kind == 1:
            u[s:e], v[s:e] = np.linspace(-1, 1, k), rng.uniform(-1, 1)
        elif kind == 2:
            u[s:e], v[s:e] = rng.uniform(-1, 1) + rng.uniform(0, 0.02, (2, k))
        else:
            u[s:e], v[s:e] = rng.uniform(1.5, 3, k), rng.uniform(-1, 1, k)
        s, kind = e, (kind + 1) % 4
    d = rng.choice(np.array([2.0, 2.01, 2.03, 3.0, 5.0]), n)        # equal and nearly equal depths
    p = np.empty(n, synth.POINT_DTYPE)
    p["x"], p["y"], p["z"] = u * d, v * d, -d
    p["rgba"] = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    m = np.array([1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, -1, 0], np.float32)
    return p, m


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
@pytest.mark.parametrize("wg", [64, 256])
@pytest.mark.parametrize("ppt", [1, 2, 4, 8, 16])
def test_scattered_and_ordered_tiles(orc, variant, wg, ppt):
    for n in (63, 30_001):
        pts, m = mixed_cloud(n, seed=ppt)
        efb, eimg = oracle_frame(orc, pts, m, W, H, variant)
        for grid in (0, 5):                                       # one tile and many tiles per workgroup
            fb, img = render_frame(upload(pts), m, W, H, variant, tune={"ppt": ppt, "wg": wg, "grid": grid})
            assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
            assert np.array_equal(img, eimg)


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
def test_scattered_chunks(orc, variant):
    pts, m = mixed_cloud(20_003, seed=3)
    efb, eimg = oracle_frame(orc, pts, m, W, H, variant)
    d = upload(pts)
    ends = [0, 1, 700, 701, 5000, 12_345, 20_003]
    tab = pcr.chunk_table([(d.data_ptr() + 16 * a, b - a) for a, b in zip(ends, ends[1:])])
    fb = pcr.alloc_fb(W, H, variant)
    pcr.fb_clear(fb, W, H, variant)
    pcr.render_chunks(tab, len(ends) - 1, m, W, H, variant, fb)
    img = pcr.resolve(fb, W, H, variant)
    assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
    assert np.array_equal(img.cpu().numpy().view(np.uint32), eimg)


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
@pytest.mark.parametrize("k", [7, 8, 9, 16, 21, 22, 64])
def test_dense_groups(orc, variant, k):
    """Rows of 64 lanes that fall into groups of k lanes to a pixel, on both
    sides of the smallest group that is collapsed and of how many are."""
    rng = np.random.default_rng(k)
    rows = 61
    n = 64 * rows + 5
    lane = np.arange(n) % 64
    order = np.stack([rng.permutation(64) for _ in range(rows + 1)]).reshape(-1)[:n]  # groups not in lane order
    group = np.where(np.arange(n) // 64 % 2 == 0, lane, order) // k
    u = -0.9 + 0.17 * group
    v = -0.9 + 0.02 * (np.arange(n) // 64)
    d = rng.choice(np.array([2.0, 2.01, 2.03, 3.0, 5.0]), n)
    pts = np.empty(n, synth.POINT_DTYPE)
    pts["x"], pts["y"], pts["z"] = u * d, v * d, -d
    pts["rgba"] = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    m = np.array([1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, -1, 0], np.float32)
    efb, eimg = oracle_frame(orc, pts, m, W, H, variant)
    for ppt in (1, 4, 8):
        fb, img = render_frame(upload(pts), m, W, H, variant, tune={"ppt": ppt})
        assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
        assert np.array_equal(img, eimg)


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
@pytest.mark.parametrize("vis", [1, 3, 4, 5, 16, 17, 63])
def test_few_visible_lanes(orc, variant, vis):
    """Rows of which `vis` lanes are visible, scattered or along a line, on both
    sides of the fewest that a tile is judged by."""
    rng = np.random.default_rng(vis)
    rows = 64
    n = 64 * rows
    u, v = rng.uniform(1.5, 3, n), rng.uniform(-1, 1, n)           # outside the view
    for r in range(rows):
        at = 64 * r + np.sort(rng.choice(64, vis, replace=False))
        if r // 8 % 2:
            u[at], v[at] = np.linspace(-0.5, 0.5, vis), rng.uniform(-1, 1)
        else:
            u[at], v[at] = rng.uniform(-1, 1, vis), rng.uniform(-1, 1, vis)
    d = rng.choice(np.array([2.0, 2.01, 2.03, 3.0, 5.0]), n)
    pts = np.empty(n, synth.POINT_DTYPE)
    pts["x"], pts["y"], pts["z"] = u * d, v * d, -d
    pts["rgba"] = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    m = np.array([1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, -1, 0], np.float32)
    efb, eimg = oracle_frame(orc, pts, m, W, H, variant)
    for ppt, grid in ((1, 0), (4, 0), (4, 3), (8, 0)):
        fb, img = render_frame(upload(pts), m, W, H, variant, tune={"ppt": ppt, "wg": 64, "grid": grid})
        assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
        assert np.array_equal(img, eimg)
