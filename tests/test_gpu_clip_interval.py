"""The interval form of the sigma clip at the ends of its register classes and where an interval
end is hard to find: stacks of 1 - 128 frames around the groups of eight and the classes, small
and large ksigma (down to everything dropped), values that tie at the threshold, ends that
cancel to nearly zero (many floats round to one difference), infinities and the largest
floats.  Keep masks equal to the FP64 oracle's except where it calls a value near its
threshold."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(rd, orc, vals, ksigma, iters, missing=False):
    dev = torch.from_numpy(np.ascontiguousarray(vals)).cuda()
    out, keep, nrej = rd.combine(dev, ksigma, iters, want_keep=True, want_nrej=True, missing=missing)
    out, keep = out.cpu().numpy().astype(np.float64), keep.cpu().numpy()
    o_out, o_keep, o_nrej, near = orc.combine(vals.astype(np.float64), ksigma, iters, missing=missing)
    near = np.broadcast_to(near.any(axis=0), keep.shape)  # one near value may change what follows in its column
    bad = (keep != o_keep) & (near == 0)
    assert not bad.any(), (vals.shape, ksigma, np.argwhere(bad)[:3])
    same = (keep == o_keep).all(axis=0)
    assert np.array_equal(np.isnan(out[same]), np.isnan(o_out[same]))
    good = same & np.isfinite(o_out)
    assert np.all(np.abs(out[good] - o_out[good]) <= 2e-6 * np.maximum(np.abs(o_out[good]), 1e-30))
    if same.all():
        assert int(nrej.cpu()[0]) == o_nrej


@pytest.mark.parametrize("N", [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 103, 104, 105, 127, 128])
def test_register_classes(orc, N):
    import paper_2008_11486_amd as rd

    rng = np.random.default_rng(N)
    vals = rng.normal(100.0, 10.0, size=(N, 7, 151)).astype(np.float32)
    vals[rng.random(vals.shape) < 0.05] += 400.0
    for ksigma, iters in ((3.0, 3), (1.5, 5), (0.3, 2), (3.0, 0)):
        _check(rd, orc, vals, ksigma, iters)
    miss = vals.copy()
    miss[rng.random(vals.shape) < 0.2] = np.nan
    _check(rd, orc, miss, 2.0, 3, missing=True)


@pytest.mark.parametrize("N", [12, 20, 40, 60, 120])
def test_hard_interval_ends(orc, N):
    import paper_2008_11486_amd as rd

    rng = np.random.default_rng(100 + N)
    w = 400
    vals = np.zeros((N, 6, w), np.float32)
    # nine tenths A, one tenth 0: m = 3 sigma, the lower end of the interval is 0 up to rounding
    A = rng.uniform(1.0, 5e4, size=(2, w)).astype(np.float32)
    vals[:, 0:2] = A
    vals[: max(1, N // 10), 0:2] = 0.0
    vals[-1, 1] = A[1] * 50  # and an outlier above
    vals[:, 2] = rng.integers(0, 4, size=(N, w))  # ties
    vals[:, 3] = rng.normal(0.0, 1e-3, size=(N, w))  # around zero
    vals[0, 3] = 1e4
    vals[:, 4] = rng.normal(0.0, 1e30, size=(N, w))
    vals[0, 4] = 3.3e38
    vals[:, 5] = 7.0
    vals[1, 5, ::2] = np.inf  # poisons its column
    for ksigma in (3.0, 1.0, 0.5):
        _check(rd, orc, vals, ksigma, 3)
