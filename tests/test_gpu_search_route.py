"""The full-window search of large problems goes through row spectra.  Against the direct sums of
the same call (which the request for score planes selects): integer offsets and flags equal,
sub-pixel offsets within 2 float ulps, peaks and runners-up to rounding, over odd and even
sizes, few and many frames, and frames that the spectra cannot settle (flat, periodic, with
missing or infinite values), whose results are the direct search's.  A workspace of the direct
search, a tuned launch shape or a small problem keeps the direct sums to the bit."""
import ctypes

import numpy as np
import pytest
import torch

from helpers import ulp32

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _no_tuned_shapes():
    """A shape that an earlier caller of this process tuned would keep the direct search."""
    import paper_2008_11486_amd as rd

    rd.tune_clear()


def _field(rng, N, W, H, R):
    big = rng.normal(1000.0, 30.0, size=(H + 2 * R, W + 2 * R)).astype(np.float32)
    at = [(0, 0)] + [tuple(rng.integers(-R, R + 1, 2)) for _ in range(N)]
    at[min(1, N)] = (R, -R)  # a maximum on the window border
    f = np.stack([big[R + dy:R + dy + H, R + dx:R + dx + W] for dx, dy in at])
    f[1:] += rng.normal(0.0, 5.0, size=f[1:].shape).astype(np.float32)
    return torch.from_numpy(f).cuda()


def _same(rd, a, b):
    for k in ("dx", "dy", "flags"):
        assert np.array_equal(a[k], b[k]), k
    for k in ("sx", "sy"):
        d = np.abs(a[k].astype(np.float64) - b[k])
        assert np.all(d <= 2 * ulp32(b[k])), k
    np.testing.assert_allclose(a["peak"], b["peak"], rtol=1e-11, equal_nan=True)
    np.testing.assert_allclose(a["second"], b["second"], rtol=1e-9, equal_nan=True)


def _direct_bytes(rd, W, H, N, R):
    """What the direct search needs, as the refusal of an 8-byte workspace states it."""
    with pytest.raises(rd.ReduceError) as e:
        t = torch.zeros((N, H, W), device="cuda")
        rd.register(t[0].contiguous(), t, R, ws=torch.empty(8, dtype=torch.uint8, device="cuda"))
    return int(str(e.value).split("needs ")[1].split()[0])


@pytest.mark.parametrize("W,H,N,R", [(512, 512, 16, 17), (401, 387, 16, 33), (1023, 1001, 5, 17), (1024, 640, 40, 9),
                                     (700, 650, 1, 65), (2051, 700, 2, 30)])
def test_routed_search_matches_direct_sums(W, H, N, R):
    import paper_2008_11486_amd as rd

    f = _field(np.random.default_rng(W + N), N, W, H, R)
    ref, frames = f[0].clone(), f[1:].clone()
    assert rd.register_ws_bytes(W, H, N, R) > _direct_bytes(rd, W, H, N, R)  # the search goes through spectra
    got = rd.offsets_to_numpy(rd.register(ref, frames, R))
    want = rd.offsets_to_numpy(rd.register(ref, frames, R, want_scores=True)[0])
    _same(rd, got, want)


def test_routed_search_of_unsettled_frames():
    import paper_2008_11486_amd as rd

    W, H, N, R = 512, 500, 16, 17
    f = _field(np.random.default_rng(9), N, W, H, R)
    ref, frames = f[0].clone(), f[1:].clone()
    frames[1] = 1000.0                                   # every score ties
    frames[2] = frames[2][:, :8].repeat(1, W // 8 + 1)[:, :W]  # periodic in x: maxima tie every 8 columns
    frames[3, 40, 50] = float("nan")
    frames[4, 3, 3] = float("nan")                       # met by some offsets only
    frames[5, 200, 100] = float("inf")
    frames[6] = 0.0
    frames[7] = frames[7] * 1e30
    got = rd.register(ref, frames, R)
    want = rd.register(ref, frames, R, want_scores=True)[0]
    for k in (1, 2, 3, 4, 5, 6):  # the fallback is the direct search itself
        assert torch.equal(got[k], want[k]), k
    ok = [0] + list(range(7, N))
    _same(rd, rd.offsets_to_numpy(got)[ok], rd.offsets_to_numpy(want)[ok])


def test_direct_sums_are_kept(tmp_path):
    import paper_2008_11486_amd as rd

    W, H, N, R = 512, 512, 16, 17
    f = _field(np.random.default_rng(3), N, W, H, R)
    ref, frames = f[0].clone(), f[1:].clone()
    want = rd.register(ref, frames, R, want_scores=True)[0]
    small = torch.empty(_direct_bytes(rd, W, H, N, R), dtype=torch.uint8, device="cuda")
    assert torch.equal(rd.register(ref, frames, R, ws=small), want)  # the workspace of the direct search
    out = torch.empty_like(want)
    if small.numel() <= int(rd.lib().reduce_register_static_max()):
        assert torch.equal(rd.register_static(ref, frames, R, out=out), want)
    try:
        rd.tune_register(ref, frames, R, reps=1)
        path = str(tmp_path / "t.json")
        rd.tune_save(path)
        tuned = rd.register(ref, frames, R, want_scores=True)[0]
        assert torch.equal(rd.register(ref, frames, R), tuned)  # a tuned shape is used by every later call
        rd.tune_clear()
        rd.tune_load(path)
        assert torch.equal(rd.register(ref, frames, R), tuned)
    finally:
        rd.tune_clear()
    centres = torch.zeros((N, 2), dtype=torch.int32, device="cuda")
    assert torch.equal(rd.register(ref, frames, R, centers=centres), want)
    few = frames[:2, :128, :128].contiguous()
    small_ref = ref[:128, :128].contiguous()
    assert torch.equal(rd.register(small_ref, few, 8), rd.register(small_ref, few, 8, want_scores=True)[0])


@pytest.mark.parametrize("ref_index", [0, 7, 11])
def test_batch_takes_the_same_route(ref_index):
    import paper_2008_11486_amd as rd

    W, H, N, R = 600, 520, 12, 20
    f = _field(np.random.default_rng(5), N - 1, W, H, R)
    raw = f.round().to(torch.int32).to(torch.int16)
    dark = torch.zeros((H, W), device="cuda")
    flat = torch.ones((H, W), device="cuda")
    batch = rd.StackBatch([(raw, dark, flat, R)], ref_index=ref_index)
    batch.run()
    offs = batch.result(0)[2]
    cal = rd.calibrate(raw, dark, flat)
    others = [k for k in range(N) if k != ref_index]
    frames = cal[others].contiguous()
    assert rd.register_ws_bytes(W, H, N - 1, R) > _direct_bytes(rd, W, H, N - 1, R)
    want = rd.offsets_to_numpy(rd.register(cal[ref_index].contiguous(), frames, R))
    assert offs[others].tobytes() == want.tobytes()
    assert (offs[ref_index]["dx"], offs[ref_index]["dy"], offs[ref_index]["peak"]) == (0, 0, 0.0)
