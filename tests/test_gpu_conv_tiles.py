"""The network's convolutions and its data gradient at the edges of their tiles (64 output columns
by eight rows forward; 64 column pairs by four row pairs backward) for odd and even image
sizes.  Against float64 sums of the stored inputs, rounded to bfloat16: a float sum of n
products is off by at most n 2^-24 of the sum of their magnitudes, and its rounding may then go
the other way, by one bfloat16 unit; at most one value in a hundred does."""
import numpy as np
import pytest

from test_gpu_learned import _net_case, bf16_ulp, rd  # noqa: F401 (rd is a fixture)

pytestmark = pytest.mark.gpu


def _forward(x, w):
    """3x3, stride 2, padding 1: x [B][H][W][Cin], w [9][Cin][32]."""
    B, H, W, c = x.shape
    Ho, Wo = (H + 1) // 2, (W + 1) // 2
    p = np.zeros((B, 2 * Ho + 1, 2 * Wo + 1, c))
    p[:, 1:H + 1, 1:W + 1] = x
    return sum(p[:, t // 3:t // 3 + 2 * Ho:2, t % 3:t % 3 + 2 * Wo:2] @ w[t] for t in range(9))


def _backward(dz, w, H, W):
    B, Ho, Wo, _ = dz.shape
    p = np.zeros((B, 2 * Ho + 1, 2 * Wo + 1, w.shape[1]))
    for t in range(9):
        p[:, t // 3:t // 3 + 2 * Ho:2, t % 3:t % 3 + 2 * Wo:2] += dz @ w[t].T
    return p[:, 1:H + 1, 1:W + 1]


def _close(got, exact, rounded, magnitude, terms, label):
    diff = np.abs(got - rounded)
    assert np.all(diff <= 1.0001 * bf16_ulp(exact) + terms * 2.0 ** -24 * magnitude + 1e-30), label
    assert np.mean(diff > 0) <= 0.01, label


@pytest.mark.parametrize("B,h,w", [(1, 16, 16), (2, 17, 257), (1, 127, 130), (2, 129, 255), (1, 35, 514)])
def test_conv_tiles(rd, orc, B, h, w):  # noqa: F811
    c = _net_case(rd, orc, B, h, w, seed=h * w)
    parts = orc.cnn_split(c["params"])

    def stored(t):
        return rd.bf16_bits_to_float(t).cpu().numpy().astype(np.float64)

    acts = [c["x"]] + [stored(c["cws"].activation(l)) for l in range(1, 5)]
    for l in range(1, 5):
        wt, b = orc.bf16_round(parts[f"w{l}"]), parts[f"b{l}"]
        y = np.maximum(_forward(acts[l - 1], wt) + b, 0.0)
        mag = _forward(np.abs(acts[l - 1]), np.abs(wt)) + np.abs(b)
        _close(acts[l], y, orc.bf16_round(y), mag, 289, f"activation {l}")
    dz1, dz2 = stored(c["cws"].grad_z(1)), stored(c["cws"].grad_z(2))
    wt = orc.bf16_round(parts["w2"])
    dx = _backward(dz2, wt, *dz1.shape[1:3]) * (acts[1] > 0)
    _close(dz1, dx, orc.bf16_round(dx), _backward(np.abs(dz2), np.abs(wt), *dz1.shape[1:3]), 128, "gradient 1")
