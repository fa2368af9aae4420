"""Which stacks of a batch the benchmark counts as searched through row spectra (CPU only: the
library's workspace queries)."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_stacks_through_row_spectra_are_told_apart():
    import paper_2008_11486_amd as rd

    spec = importlib.util.spec_from_file_location("bench_route_under_test", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    rd.tune_clear()
    b = 4096  # never read

    def stack(N, W, H, R, search=0):
        return rd.StackDesc(b, W, W * H, b, b, W, W, H, N, 0, R, 3, 3.0, 0, b, b, b, b, 0, 0, search, 0)

    class Batch:
        descs = (rd.StackDesc * 6)(stack(10, 1024, 1000, 21), stack(4, 512, 512, 17), stack(4, 512, 512, 17, 1),
                                   stack(1, 1024, 1000, 21), stack(10, 9000, 600, 21), stack(5, 512, 512, 0))

    assert bench.spectral_stacks(rd, Batch) == [True, False, True, False, False, False]
    assert [d.search for d in Batch.descs] == [0, 0, 1, 0, 0, 0]
