"""Windows of up to 5 x 5 candidates (four template columns per lane, straight from global
memory) against the sums in NumPy float64: templates narrower than a lane's four columns, at
and around the edges of a lane, of a tile of columns, of a wave's rows and of a tile of rows;
one to more slots than a group of eight tiles; centres inside the clip and on its rim, where
columns and rows are clamped.  Nothing outside the template's reach is weighed, not even by
zero: it is NaN here where every candidate lies inside the frame.

A sum of n products in a tree of depth at most 4 * 60 + 6 + 4 + tiles / 8 is off by at most that
many ulps of the sum of magnitudes; the mean's own rounding adds as much again: 1e-12 of it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [0, 1, 2])
@pytest.mark.parametrize("tw,th,N", [(1, 1, 1), (3, 7, 2), (4, 3, 1), (5, 59, 3), (255, 61, 2), (256, 240, 9),
                                     (257, 241, 4), (1030, 500, 3), (2301, 16, 2)])
def test_small_window_scores(R, tw, th, N):
    import paper_2008_11486_amd as rd

    rng = np.random.default_rng(100 * tw + th + R)
    Rmax = R + 3
    x0, y0 = Rmax + int(rng.integers(0, 4)), Rmax + int(rng.integers(0, 4))
    W, H = x0 + tw + Rmax + int(rng.integers(0, 5)), y0 + th + Rmax + int(rng.integers(0, 5))
    ref = rng.normal(500.0, 40.0, size=(H, W)).astype(np.float32)
    frames = rng.normal(500.0, 40.0, size=(N, H, W)).astype(np.float32)
    centres = rng.integers(-Rmax, Rmax + 1, size=(N, 2)).astype(np.int32)
    centres[0] = (-Rmax, Rmax)
    if N > 1:
        centres[1] = (1, -1)
        reach = np.zeros((H, W), bool)
        reach[y0 - 1 - R:y0 + th - 1 + R, x0 + 1 - R:x0 + tw + 1 + R] = True
        frames[1][~reach] = np.nan
    _, got = rd.register(torch.from_numpy(ref).cuda(), torch.from_numpy(frames).cuda(), R, Rmax,
                         centers=torch.from_numpy(centres).cuda(), tmpl=(x0, y0, tw, th), want_scores=True)
    got = got.cpu().numpy()
    t = ref[y0:y0 + th, x0:x0 + tw].astype(np.float64)
    mean = t.mean()
    for k in range(N):
        for j in range(2 * R + 1):
            for i in range(2 * R + 1):
                dx, dy = int(centres[k, 0]) - R + i, int(centres[k, 1]) - R + j
                if max(abs(dx), abs(dy)) > Rmax:
                    assert got[k, j, i] == -np.inf
                    continue
                f = frames[k, y0 + dy:y0 + dy + th, x0 + dx:x0 + dx + tw].astype(np.float64)
                tol = 1e-12 * float(((np.abs(t) + abs(mean)) * np.abs(f)).sum())
                assert abs(got[k, j, i] - float(((t - mean) * f).sum())) <= tol, (k, dx, dy)
