"""The batched call settles each stack's search once, whatever another thread does to the tuner's
table while the call runs: between its layout and its launches (here, during the upload of its
descriptors) a tuned shape comes or goes, and the launches stay those of the layout.  Host
side only, with recorded launches."""
import launch_recorder

SETUP = """
    b = 1 << 40  # never read
    W, H, N, R = 1024, 1000, 9, 21
    def stack(W, H, N, R):
        return rd.StackDesc(b, W, W * H, b, b, W, W, H, N, 2, R, 3, 3.0, 0, b, b, b, b, 0, 0, 0, 0)
    arr = (rd.StackDesc * 2)(stack(W, H, N, R), stack(W, H, N, R))
    f = rd.register_plan(W, H, N, R)
    line = ('{{"arch": "%s", "op": "register", "W": %d, "H": %d, "R": %d, "Rmax": %d, "K": %d, "G": %d, "S": %d, '
            '"TY": %d, "CPT": %d, "ms": 1.0}}')
    shape = (W, H, R, R, f["K"], f["G"], f["S"], f["TY"], {rows} * f["BR"] // f["TY"])
    path = {path!r}
    with open(path, "w") as t:  # entries of other devices are skipped; without one the name is "unknown"
        t.write("".join(line % ((arch,) + shape) + chr(10) for arch in ("unknown", "gfx950")))
    def call():
        assert L.reduce_stack_batch(arr, 2, ctypes.c_void_p(b), 1 << 40, None) == rd.OK, L.reduce_last_error()
        return launches()
    untuned = call()
    rd.tune_load(path)
    tuned = call()
    assert count(untuned, "spec_cols") == 2 and count(untuned, "batch_score") == 0, untuned
    assert count(tuned, "spec_cols") == 0 and count(tuned, "batch_score") == 1, tuned
"""


def test_a_shape_tuned_during_the_call_changes_nothing(tmp_path):
    # the same plan, so that only the route differs; and a taller tile, so that the fallback's plan would
    for rows in (1, 2):
        launch_recorder.run(tmp_path, SETUP.format(path=str(tmp_path / "t.json"), rows=rows) + """
    rd.tune_clear()
    hook = COPY(lambda: rd.tune_load(path))
    rec.rec_on_copy(hook)
    assert call() == untuned
    """)


def test_a_table_cleared_during_the_call_changes_nothing(tmp_path):
    launch_recorder.run(tmp_path, SETUP.format(path=str(tmp_path / "t.json"), rows=1) + """
    hook = COPY(rd.tune_clear)
    rec.rec_on_copy(hook)
    assert call() == tuned
    """)


def test_a_workspace_of_the_direct_sums_is_accepted(tmp_path):
    launch_recorder.run(tmp_path, SETUP.format(path=str(tmp_path / "t.json"), rows=1) + """
    direct = int(L.reduce_stack_batch_ws(arr, 2))  # with the tuned shape
    rd.tune_clear()
    assert direct < int(L.reduce_stack_batch_ws(arr, 2))
    assert L.reduce_stack_batch(arr, 2, ctypes.c_void_p(b), direct, None) == rd.OK, L.reduce_last_error()
    assert launches() == tuned
    assert L.reduce_stack_batch(arr, 2, ctypes.c_void_p(b), direct - 1, None) == rd.ERR_WORKSPACE
    assert str(direct).encode() in L.reduce_last_error() and launches() == []
    arr[1].search = 1  # asked for: its workspace is needed
    assert L.reduce_stack_batch(arr, 2, ctypes.c_void_p(b), direct, None) == rd.ERR_WORKSPACE
    """)
