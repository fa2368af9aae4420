"""The network's input, bit for bit: every value is the double asinh of the standardised block
mean, rounded to float and then to bfloat16, though most are evaluated in float within an
interval that decides the roundings.  Against NumPy on the block means, the mean and the
sigma that the call leaves in its workspace: values from a billionth of sigma to thousands of it,
block means equal to each other (sigma zero) and counts that are no multiple of four."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _bf16(x):
    u = x.astype(np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


@pytest.mark.parametrize("W,H,N,spread", [(1024, 1024, 2, 1.0), (1024, 1024, 1, 8.0), (404, 396, 3, 4.0),
                                          (20, 28, 2, 1.0), (64, 64, 1, 0.0)])
def test_network_input_bits(W, H, N, spread):
    import paper_2008_11486_amd as rd

    rng = np.random.default_rng(W + N)
    f = rng.normal(size=(N, H, W)) * np.exp(spread * rng.normal(size=(N, H, W))) if spread else np.full((N, H, W), 3.0)
    ws = torch.empty(rd.cnn_input_ws_bytes(W, H, N), dtype=torch.uint8, device="cuda")
    got = rd.cnn_input(torch.from_numpy(f.astype(np.float32)).cuda(), ws=ws)
    bits = got.view(torch.int16).cpu().numpy().view(np.uint16).reshape(N, -1)
    raw = ws.cpu().numpy()
    n = (W // 4) * (H // 4)

    def al(b):
        return (b + 255) // 256 * 256

    at = al(4 * n * N) + al(16 * ((n + 255) // 256) * N)
    m = raw[:4 * n * N].view(np.float32).reshape(N, n).astype(np.float64)
    mean = raw[at + al(8 * N):][:8 * N].view(np.float64)
    sd = raw[at + 2 * al(8 * N):][:8 * N].view(np.float64)
    for k in range(N):
        np.testing.assert_allclose(mean[k], m[k].mean(), rtol=1e-5, atol=1e-5 * np.abs(m[k]).max())
        z = (m[k] - mean[k]) / sd[k] if sd[k] > 0 else np.zeros(n)
        assert np.array_equal(bits[k], _bf16(np.arcsinh(z))), k
