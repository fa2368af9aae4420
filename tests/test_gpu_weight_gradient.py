"""Weight and bias gradients of the input layer and of a 32-channel layer where the strips of
64 output pixels end in a remainder, a group walks over several strips, or the frame is the
smallest: against FP64 sums over the GPU's own activations and gradient planes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _wgrad64(x, dz):
    """x [B][H][W][ci], dz [B][Ho][Wo][co] float64 -> sums [9][ci][co] of x * dz and of |x| |dz|."""
    B, Ho, Wo, _ = dz.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 2, 1, 2))
    out = []
    for a, b in ((xp, dz), (xp.abs(), dz.abs())):
        b2 = b.reshape(-1, b.shape[-1])
        out.append(torch.stack([a[:, ky:ky + 2 * Ho:2, kx:kx + 2 * Wo:2].reshape(-1, a.shape[-1]).t() @ b2
                                for ky in range(3) for kx in range(3)]))
    return out


@pytest.mark.parametrize("B,h,w", [(1, 16, 16), (2, 37, 259), (1, 301, 130), (3, 640, 517)])
def test_weight_gradients_of_ragged_strips(B, h, w):
    import paper_2008_11486_amd as rd
    from paper_2008_11486_amd import learned

    rng = np.random.default_rng(B * 1000 + w)
    params = torch.from_numpy(learned.init_params(3) + rng.normal(0, 0.05, rd.cnn_num_params()).astype(np.float32))
    inp = torch.from_numpy(rng.normal(size=(2 * B, h, w)).astype(np.float32)).bfloat16()
    bits = inp.view(torch.int16).cuda()
    cws = rd.CnnWorkspace(B, h, w)
    pd = params.cuda()
    pred = rd.cnn_forward(bits[:B], bits[B:], pd, cws, ref_shared=False)
    target = torch.from_numpy(rng.normal(size=(B, 2)).astype(np.float32)).cuda()
    _, grad = rd.cnn_backward(bits[:B], bits[B:], pd, pred, target, cws, ref_shared=False)
    grad = grad.cpu().double()
    at = learned.param_slices()
    x = torch.stack([inp[:B].double(), inp[B:].double()], dim=-1)
    for layer in (1, 2):
        dz = rd.bf16_bits_to_float(cws.grad_z(layer)).cpu().double()
        want, mag = _wgrad64(x, dz)
        # a sum passes through at most 64 additions per strip row of its group (the walk of
        # one of 4 groups of up to 256 workgroups) and 64 more over groups and workgroups
        steps = B * -(-dz.shape[2] // 64) * dz.shape[1]
        per = -(-steps // (4 * min(256, -(-steps // 4))))
        unit = 2.0 ** -24 * (64 * per + 64)
        got = grad[at["w%d" % layer][0]].view(at["w%d" % layer][1])
        assert ((got - want).abs() <= unit * mag).all(), layer
        gb = grad[at["b%d" % layer][0]]
        assert ((gb - dz.sum((0, 1, 2))).abs() <= unit * dz.abs().sum((0, 1, 2))).all(), layer
        x = rd.bf16_bits_to_float(cws.activation(layer)).cpu().double()
