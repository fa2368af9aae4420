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
