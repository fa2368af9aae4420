"""The one-pass spline shift where its strips of 64 columns, batches of 32 rows and cut walks end:
frames of one and two rows or columns, lines shorter than the recursions' warm-up, one row or
column more than a tile, outputs at positions clamped far outside the frame, and enough frames
that walks are not cut.  Against the FP64 oracle, within what single precision can do next to
the frame's brightest value M: a line's second derivatives reach 12 M (24 M of second
differences over the smallest row sum 2 of the (1, 4, 1) system), a value takes at most
(1 + 2 * 0.065 * 12) M < 2.6 M of terms, each through about ten roundings, in two passes:
2 * 10 * 2.6 * 2^-24 M < 3.2e-6 M."""
import numpy as np
import pytest
import torch

from oracle import spline as orc_spline

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 0.3), (2, 1, 70, 0.4), (2, 70, 1, 0.4), (2, 2, 3, 0.5), (3, 5, 130, 2.0), (2, 17, 17, 3.0),
         (2, 18, 66, 1.5), (2, 33, 64, 6.0), (1, 65, 63, 5.0), (2, 96, 129, 20.0), (2, 100, 200, 90.0),
         (3, 131, 70, 300.0), (1, 200, 333, 17.4), (400, 40, 190, 4.0)]


@pytest.mark.parametrize("N,H,W,bound", CASES)
def test_strip_and_batch_ends(N, H, W, bound):
    import paper_2008_11486_amd as rd

    rng = np.random.default_rng(H * 1000 + W)
    f = (1000.0 + rng.normal(0.0, 30.0, size=(N, H, W))).astype(np.float32)
    f[:, H // 2, W // 2] += 2e4
    s = rng.uniform(-bound, bound, size=(N, 2)).astype(np.float32)
    s[0] = np.float32(bound)
    if N > 2:
        s[1] = -np.float32(bound)
        s[2] = np.round(s[2])
    x0, y0 = min(1, W - 1), 0
    for rect in ((0, 0, W, H), (x0, y0, W - x0, max(1, H - 2))):  # positions past the frame are clamped
        out = rd.shift_spline(torch.from_numpy(f).cuda(), torch.from_numpy(s).cuda(), rect).cpu().numpy()
        pick = list(range(min(N, 4))) + ([N - 1] if N > 4 else [])
        want = orc_spline.shift_spline(f[pick], s[pick], rect)

        err = np.abs(out[pick] - want).max() / np.abs(f[pick]).max()
        assert err <= 3.2e-6, (rect, err)
