"""The narrowed search's rounds on the device (sum, pick and move in one launch for windows of at
most 64 candidates, by themselves for larger ones) against the same decisions taken on the host, byte for byte:
windows on both sides of 64 candidates, no moves and several, most frames flagged and few."""
import numpy as np
import pytest
import torch

from test_gpu_learned import _host_flow, random_params, rd  # noqa: F401 (rd is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r,moves,scale", [(0, 3, 0.2), (1, 0, 0.2), (2, 2, 0.02), (3, 5, 0.2), (4, 2, 0.2), (6, 1, 0.02)])
def test_window_moves(rd, orc, r, moves, scale):  # noqa: F811
    from paper_2008_11486_amd import learned

    W, rmax, N = 256, 12, 7
    frames, _ = learned.render_stack(11, N + 1, W, W, rmax - 2)
    ref, rest = frames[0].contiguous(), frames[1:].contiguous()
    p = (random_params(orc, np.random.default_rng(r)) * scale).astype(np.float32)
    dev, centres, info = rd.propose(ref, rest, torch.from_numpy(p).cuda(), radius_max=rmax, refine_radius=r,
                                    max_moves=moves)
    want, c_host, fb, n_moves = _host_flow(rd, learned, p, ref, rest, rmax, r=r, moves=moves)
    info = info.cpu().numpy()
    np.testing.assert_array_equal(centres.cpu().numpy(), c_host)
    np.testing.assert_array_equal(info & 255, n_moves)
    np.testing.assert_array_equal((info >> 8) & 3 != 0, fb)
    assert rd.offsets_to_numpy(dev).tobytes() == want.tobytes()
