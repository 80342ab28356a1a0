"""What the autotuner searches: the launches that a schedule shapes, with both
block sizes by name (0 leaves the size to the launch, so it would time one of
them twice).  2-D passes that no schedule changes (wave passes along axes of 81,
243 and 729 nodes) keep the schedule they had.  Images that run whole FP64 solves
in one block still have schedules, for the solves that run the passes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _tuned(shape, precision, tensor=False):
    from paper_1004_1122_amd import lshom
    phase = (np.random.default_rng(sum(shape)).random(shape) < 0.4).astype(np.uint8)
    d = len(shape)
    s = lshom.Solver(phase, np.stack([np.eye(d), 5.0 * np.eye(d)]) if tensor else [1.0, 5.0])
    before = s.get_schedule(precision)
    after = s.autotune(precision=precision, reps=2)
    assert after.pop("ms_per_iter") > 0
    before.pop("ms_per_iter")
    return before, after


ROW, COL = ("rows_per_block", "row_split", "threads_row"), ("tile0", "tile1", "threads_col")


@pytest.mark.parametrize("shape,precision", [((81, 81), 0), ((81, 81), 1), ((81, 243), 0), ((729, 81), 1)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_keeps_what_no_launch_reads(shape, precision):
    before, after = _tuned(shape, precision)
    assert after == before


@pytest.mark.parametrize("shape,precision,tensor,row,col",
                         [((60, 100), 0, False, True, True), ((45, 60), 1, False, True, True),
                          ((100, 75), 1, False, True, True), ((30, 24, 20), 0, False, True, True),
                          ((81, 60), 0, False, True, False), ((60, 81), 1, False, False, True),
                          ((45, 81), 0, True, True, True), ((45, 27), 0, False, True, True),
                          ((27, 27, 27), 0, False, True, True), ((27, 27, 27), 1, False, True, True)],
                         ids=["60x100", "45x60-mixed", "100x75-mixed", "30x24x20", "81x60", "60x81-mixed",
                              "45x81-tensors", "45x27", "27x27x27", "27x27x27-mixed"])
def test_searches_both_block_sizes(shape, precision, tensor, row, col):
    before, after = _tuned(shape, precision, tensor)
    for tuned, keys, axis in ((row, ROW, len(shape) - 1), (col, COL, 0)):
        if tuned:
            assert after[keys[2]] in (128, 256)
        else:
            assert all(after[k] == before[k] for k in keys) and after["radix"][axis] == before["radix"][axis]


def test_small_images_use_the_schedule_where_they_run_the_passes():
    from paper_1004_1122_amd import lshom
    phase = (np.random.default_rng(4).random((45, 63)) < 0.4).astype(np.uint8)
    s = lshom.Solver(phase, [1.0, 9.0])
    forms = [dict(), dict(method=lshom.METHOD_PIPECG), dict(history=50), dict(precision=1)]
    first = [s.solve((1.0, 0.2), tol=1e-8, **kw) for kw in forms]
    for p in (0, 1):
        s.set_schedule(dict(s.get_schedule(p), radix=[[3, 3, 5], [3, 7, 3]], rows_per_block=6))
    for k, kw in enumerate(forms):
        e, _, info = s.solve((1.0, 0.2), tol=1e-8, **kw)
        assert info["iterations"] == first[k][2]["iterations"]
        assert float((e - first[k][0]).norm() / e.norm()) < (1e-7 if kw.get("precision") else 1e-10)
        assert not torch.equal(e, first[k][0])
