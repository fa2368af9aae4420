"""Counts of dropped values of the batched call: stacks of 4096 and more tiles of 64 x 4 pixels add
into counters of their own that are summed after the fused phase."""
import numpy as np
import pytest
import torch

from test_gpu_batch import rd, stagewise  # noqa: F401 (rd is a fixture)

pytestmark = pytest.mark.gpu

LARGE = (12, 1100, 1030)  # 18 x 258 tiles
SMALL = (13, 150, 90)


def _stack(rng, N, W, H, mask=None):
    raw = rng.normal(1000.0, 30.0, size=(N, H, W))
    raw[rng.random(size=raw.shape) < 2e-3] += 9000.0
    raw = torch.from_numpy(raw.round().astype(np.int16)).cuda()
    dark, flat = torch.zeros((H, W), device="cuda"), torch.ones((H, W), device="cuda")
    if mask is not None:
        mask = torch.from_numpy((rng.random(size=(H, W)) < mask).astype(np.uint8)).cuda()
    return raw, dark, flat, 1, None, mask


def test_stacks_that_share_a_counter_get_their_sum(rd):  # noqa: F811
    rng = np.random.default_rng(31)
    stacks = [_stack(rng, *size) for size in (LARGE, SMALL, LARGE, LARGE)]
    own = rd.StackBatch(stacks)
    own.run()
    counts = [own.result(i)[3] for i in range(4)]
    assert min(counts) > 0
    shared = rd.StackBatch(stacks)
    total = torch.full((1,), -7, dtype=torch.int64, device="cuda")
    for i in range(4):
        shared.descs[i].n_rej = total.data_ptr()
    for _ in range(2):
        shared.run()
        assert int(total.cpu()[0]) == sum(counts)


def test_counts_of_masked_stacks_on_a_reused_workspace(rd):  # noqa: F811
    rng = np.random.default_rng(32)
    stacks = [_stack(rng, *size, mask=0.02) for size in (LARGE, SMALL)]
    batch = rd.StackBatch(stacks)
    for _ in range(2):
        batch.run()
        for i, (raw, dark, flat, R, _, mask) in enumerate(stacks):
            img, rect, offs, nrej = batch.result(i)
            want_img, want_rect, want_offs, want_nrej = stagewise(rd, raw, dark, flat, R, mask=mask)
            assert nrej == want_nrej > 0, i
            assert np.array_equal(rect, want_rect) and offs.tobytes() == want_offs.tobytes(), i
            assert np.array_equal(img.cpu().numpy(), want_img, equal_nan=True), i
        for s in stacks:  # other frames and other hits in the same buffers
            s[0].copy_(s[0].flip(0, 1) + 3)


def test_unsettled_frames_around_the_reference_take_the_direct_search(rd):  # noqa: F811
    N, W, H, R = 9, 300, 260, 9
    rng = np.random.default_rng(33)
    big = rng.normal(1000.0, 30.0, size=(H + 2 * R, W + 2 * R))
    at = rng.integers(-R + 1, R, size=(N, 2))
    raw = np.stack([big[R + y:R + y + H, R + x:R + x + W] for x, y in at]) + rng.normal(0.0, 5.0, (N, H, W))
    raw[[0, 3, 8]] = 1000.0  # every score ties: the spectra settle nothing
    raw = torch.from_numpy(raw.round().astype(np.int16)).cuda()
    dark, flat = torch.zeros((H, W), device="cuda"), torch.ones((H, W), device="cuda")
    cal = rd.calibrate(raw, dark, flat)
    for ref in (2, 5, 7):
        batch = rd.StackBatch([(raw, dark, flat, R)], ref_index=ref, search="spectral")
        batch.run()
        offs = batch.result(0)[2]
        others = [k for k in range(N) if k != ref]
        want = rd.offsets_to_numpy(rd.register(cal[ref].contiguous(), cal[others].contiguous(), R, want_scores=True)[0])
        for i, k in enumerate(others):
            if k in (0, 3, 8):
                assert offs[k].tobytes() == want[i].tobytes(), (ref, k)
            else:
                assert (offs[k]["dx"], offs[k]["dy"]) == (want[i]["dx"], want[i]["dy"]), (ref, k)
