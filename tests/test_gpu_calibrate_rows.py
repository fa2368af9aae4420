"""Calibration of rows of every length modulo 8 and every start and pitch modulo 16 bytes (odd
elements among them), shorter than 8 pixels too, and frame counts around the frames loaded
ahead: to the bit the float32 operations of numpy, with nothing written past the frames."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("W", [1, 7, 8, 9, 12, 15, 16, 23, 33, 250, 1021])
def test_rows_of_any_start_and_pitch(W, bias):
    import ctypes

    import paper_2008_11486_amd as rd

    L = rd.lib()
    rng = np.random.default_rng(W)
    p = lambda t, o=0: ctypes.c_void_p(t.data_ptr() + o)  # noqa: E731
    for H, N, lead, pad, cal_pad in ((5, 1, 0, 0, 0), (3, 4, 1, 50, 1), (4, 5, 3, 7, 3), (2, 9, 6, 1, 2)):
        rp, cp = W + pad, W + cal_pad
        raw = rng.integers(0, 65536, lead + N * H * rp + 1, dtype=np.uint16)
        cal = [rng.uniform(lo, hi, lead + H * cp).astype(np.float32) for lo, hi in ((200, 300), (50, 150), (0.9, 1.1))]
        dev = torch.from_numpy(raw.view(np.int16)).cuda()
        cals = [torch.from_numpy(c).cuda() for c in cal]
        out = torch.full((N * H * W + 16 + lead,), -7.0, device="cuda")
        rc = L.reduce_calibrate(p(dev, 2 * lead), rp, rp * H, p(cals[0], 4 * lead) if bias else None, p(cals[1], 4 * lead),
                                p(cals[2], 4 * lead), cp, p(out, 4 * lead), W, H, N, None)
        assert rc == rd.OK
        torch.cuda.synchronize()
        r = raw[lead:lead + N * H * rp].reshape(N, H, rp)[:, :, :W].astype(np.float32)
        b, d, f = (c[lead:lead + H * cp].reshape(H, cp)[:, :W] for c in cal)
        want = ((r - b if bias else r) - d) / f
        got = out.cpu().numpy()
        assert np.array_equal(got[lead:lead + N * H * W].reshape(N, H, W), want), (H, N, lead)
        assert (got[:lead] == -7).all() and (got[lead + N * H * W:] == -7).all()
