"""Chunk tables on both sides of the size up to which the render workgroups
find their own first chunk: frames equal the flat render of the kept points."""
import numpy as np
import pytest

from gpu_util import oracle_frame, read_fb, assert_same_fb, upload
from paper_2104_07526_amd import pcr, synth

pytestmark = pytest.mark.gpu

W, H = 320, 240


def frames(variant, sizes, seed, tune=None):
    """(chunked framebuffer, kept host points): chunks of the given sizes, of
    which about a tenth each are skipped (NULL or misaligned pointer)."""
    import torch
    rng = np.random.default_rng(seed)
    pts = synth.terrain(int(sizes.sum()) + 1, seed=11)
    whole = upload(pts)
    offs = np.concatenate([[0], np.cumsum(sizes)])
    kind = rng.integers(0, 12, len(sizes))
    kind[sizes > 100_000] = 5
    rows, kept = [], []
    for c, k in enumerate(kind):
        addr = whole.data_ptr() + 16 * int(offs[c])
        rows.append((0 if k == 0 else addr + 8 if k == 1 else addr, int(sizes[c])))
        if k > 1:
            kept.append(pts[offs[c]:offs[c + 1]])
    m = synth.terrain_oblique(W, H)
    fb = pcr.alloc_fb(W, H, variant)
    pcr.fb_clear(fb, W, H, variant)
    pcr.render_chunks(pcr.chunk_table(rows), len(rows), m, W, H, variant, fb, tune=tune)
    torch.cuda.synchronize()
    return fb, np.concatenate(kept + [pts[:0]]), m


@pytest.mark.parametrize("variant", [pcr.BASIC, pcr.DEDUP, pcr.HQ])
@pytest.mark.parametrize("nchunks", [1, 63, 64, 65, 2047, 2048, 2049])
def test_table_sizes(orc, variant, nchunks):
    sizes = np.random.default_rng(nchunks).integers(0, 600, nchunks)
    sizes[: nchunks // 3] = 0                                     # a run of chunks without a tile
    fb, kept, m = frames(variant, sizes, nchunks)
    efb, _ = oracle_frame(orc, kept, m, W, H, variant)
    assert_same_fb(read_fb(fb, W, H, variant), efb, variant)


@pytest.mark.parametrize("variant", [pcr.DEDUP, pcr.HQ])
def test_more_tiles_than_workgroups(orc, variant):
    """64-point tiles, more of them than the launch has workgroups: each takes
    a range that crosses chunks."""
    sizes = np.concatenate([np.random.default_rng(1).integers(0, 9000, 1500), [3_000_001]])
    fb, kept, m = frames(variant, sizes, 1, tune={"ppt": 1, "wg": 64})
    assert len(kept) > 64 * (1 << 17)
    efb, _ = oracle_frame(orc, kept, m, W, H, variant)
    assert_same_fb(read_fb(fb, W, H, variant), efb, variant)
