"""A batch whose workspace holds the direct sums only: the stacks that row spectra would search by
themselves are searched directly, with the bits of the direct search of the same frames."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_batch_in_the_workspace_of_the_direct_sums():
    import paper_2008_11486_amd as rd

    rd.tune_clear()
    rng = np.random.default_rng(21)
    stacks = []
    for W, H, N, R in ((600, 520, 12, 20), (130, 90, 5, 4)):
        big = rng.normal(1000.0, 30.0, size=(H + 2 * R, W + 2 * R))
        at = rng.integers(-R + 1, R, size=(N, 2))
        raw = np.stack([big[R + y:R + y + H, R + x:R + x + W] for x, y in at]) + rng.normal(0.0, 5.0, (N, H, W))
        stacks.append((torch.from_numpy(raw.round().astype(np.int16)).cuda(), torch.zeros((H, W), device="cuda"),
                       torch.ones((H, W), device="cuda"), R))
    L = rd.lib()
    batch = rd.StackBatch(stacks, ref_index=3)
    assert L.reduce_stack_batch(batch.descs, 2, 256, 8, None) == rd.ERR_WORKSPACE
    need = int(L.reduce_last_error().decode().split("needs ")[1].split()[0])
    assert need < batch.ws_bytes()
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert L.reduce_stack_batch(batch.descs, 2, ws.data_ptr(), need, stream) == rd.OK
    got = [(batch.result(i)[2], batch.result(i)[0].clone()) for i in range(2)]
    batch.run()
    for i, (raw, dark, flat, R) in enumerate(stacks):
        cal = rd.calibrate(raw, dark, flat)
        others = [k for k in range(raw.shape[0]) if k != 3]
        want, _ = rd.register(cal[3].contiguous(), cal[others].contiguous(), R, want_scores=True)  # direct sums
        assert got[i][0][others].tobytes() == rd.offsets_to_numpy(want).tobytes(), i
        assert torch.equal(got[i][1], batch.result(i)[0]), i  # the spectral route's image
