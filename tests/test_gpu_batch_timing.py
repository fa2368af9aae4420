"""Kernel timing of the batched call: a phase that launches nothing has no launch on record."""
import pytest
import torch

from test_gpu_batch import rd  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,fused", [(5, 1), (50, 0)])
def test_fused_phase_is_on_record_where_it_runs(rd, N, fused):  # noqa: F811
    raw = torch.full((N, 40, 60), 1000, dtype=torch.int16, device="cuda")
    batch = rd.StackBatch([(raw, torch.zeros((40, 60), device="cuda"), torch.ones((40, 60), device="cuda"), 1)])
    rd.prof_enable(True)
    try:
        batch.run()
        torch.cuda.synchronize()
        assert rd.prof_query("batch_fused")[1] == fused
    finally:
        rd.prof_enable(False)
