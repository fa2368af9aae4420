"""The block transforms along y of the search through row spectra, where their blocks, bands and
lag passes end: templates of one row, of exactly one block, one row more and a ragged last
block, windows of one lag pass at its widest (143 lags), of two and of three, and a narrow
frame of few spectrum columns.  Scores within the rounding bound of the FP64 oracle's direct
sums, offsets and flags equal."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (R, N, W, H): template rows th = H - 2R, blocks of M = 257 - lags of a pass
# and the row transform at every length, with odd and even widths and row starts
CASES = [(4, 2, w, 24) for w in (60, 128, 255, 512, 1001, 2048, 4095, 8192)] + [(5, 2, 513, 25)] + [
         (1, 2, 64, 3),        # th = 1
         (8, 2, 70, 256),      # M = 240, th = M
         (8, 3, 70, 257),      # th = M + 1
         (17, 2, 96, 700),     # three blocks, the last ragged
         (71, 2, 200, 400),    # 143 lags in one pass
         (72, 2, 200, 400),    # two passes of 73 lags
         (150, 2, 320, 340)]   # three passes of 101


@pytest.mark.parametrize("R,N,W,H", CASES)
def test_block_contraction_ends(orc, R, N, W, H):
    import paper_2008_11486_amd as rd

    rng = np.random.default_rng(R * 1000 + H)
    base = rng.normal(1000.0, 30.0, size=(H + 2 * R, W + 2 * R))
    frames = np.stack([base[R + dy:R + dy + H, R + dx:R + dx + W] + rng.normal(0.0, 3.0, size=(H, W))
                       for dx, dy in [(0, 0)] + [tuple(rng.integers(-R, R + 1, 2)) for _ in range(N - 1)]])
    f32 = torch.from_numpy(frames.astype(np.float32)).cuda()
    out, S = rd.register_fft(f32[0].contiguous(), f32, R, want_scores=True)
    g = rd.offsets_to_numpy(out)
    f64 = f32.cpu().numpy().astype(np.float64)
    o, So = orc.register(f64[0], f64, R, want_scores=True)
    P = max(64, 1 << (W - 1).bit_length())
    lags = -(-(2 * R + 1) // -(-(2 * R + 1) // 144))
    M = 257 - lags
    th = H - 2 * R
    t = f64[0, R:H - R, R:W - R]
    unit = 4 * 2.0 ** -53 * (10 * math.log2(P // 2) + -(-256 // M) * (124 + -(-th // M)) + P + 50)
    bound = unit * np.linalg.norm(t - t.mean()) * np.linalg.norm(f64.reshape(N, -1), axis=1)
    err = np.abs(S.cpu().numpy() - So).reshape(N, -1).max(axis=1)
    assert np.all(err <= bound), (err, bound)
    assert np.array_equal(g["dx"], o["dx"]) and np.array_equal(g["dy"], o["dy"])
    assert np.array_equal(g["flags"], o["flags"])
