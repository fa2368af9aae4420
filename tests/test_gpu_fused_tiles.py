"""Shift, bad-pixel mask and clip in one pass (stacks of up to 48 frames, tiles of 64 x 4 output
pixels) against the stage-wise chain, bit for bit: the frame counts at the ends of the three
classes, overlaps at and around a multiple of the tile, odd widths, maps that are dense
enough to leave columns with few values or none, integer and bilinear shifts."""
import numpy as np
import pytest

from helpers import to_dev
from test_gpu_batch import _make, rd, stagewise  # noqa: F401 (rd is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("density", [None, 0.01, 0.4])
def test_fused_tiles(rd, density):  # noqa: F811
    rng = np.random.default_rng(7)
    specs = [(1, 65, 9, 0, False), (2, 72, 40, 2, False), (16, 139, 70, 5, False), (17, 96, 81, 4, True),
             (32, 131, 64, 1, False), (33, 64, 64, 0, False), (48, 203, 37, 6, False), (3, 80, 30, 3, True)]
    dev = []
    for i, (N, W, H, R, _) in enumerate(specs):
        st = _make(50 + i, N, W, H, R, True, seed=8)
        mask = None if density is None else to_dev((rng.random(size=(H, W)) < density).astype(np.uint8))
        dev.append((to_dev(st.raw), to_dev(st.dark), to_dev(st.flat), R, None, mask))
    batch = rd.StackBatch(dev, integer_mode=[sp[4] for sp in specs])
    batch.run()
    for i, ((raw, dark, flat, R, _, mask), sp) in enumerate(zip(dev, specs)):
        img, rect, offs, nrej = batch.result(i)
        ref_img, ref_rect, ref_offs, ref_nrej = stagewise(rd, raw, dark, flat, R, integer_mode=sp[4], mask=mask)
        assert np.array_equal(rect, ref_rect), i
        assert np.array_equal(img.cpu().numpy(), ref_img, equal_nan=True), i
        assert offs.tobytes() == ref_offs.tobytes() and nrej == ref_nrej, i
