"""A schedule registered between two runs of a batch takes effect in the
second: its fields are, bit for bit, those of a new solver that had the
schedule from the start (the grid runs the block passes, whose rounding the
radix order changes)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("precision", [0, 1])
def test_batch_takes_a_new_schedule(precision):
    from paper_1004_1122_amd import lshom
    rng = np.random.default_rng(5)
    probs = [dict(phase=rng.integers(0, 2, size=(72, 90)).astype(np.uint8), cond=[1.0, 30.0], E=(1.0, 0.4), tol=0.0,
                  want_field=True) for _ in range(3)]
    s = lshom.Solver(probs[0]["phase"], probs[0]["cond"])
    base = s.get_schedule(precision)
    other = dict(base, radix=[r[::-1] for r in base["radix"]], rows_per_block=4)
    assert other["radix"] != base["radix"]

    def run(b):
        f, _, _ = b.run(precision=precision, max_iter=40, allow_fail=True)
        return [x.clone() for x in f]

    def solver(sched):
        b = lshom.BatchSolver()
        if sched:
            b.set_schedule(sched)
        b.prepare(probs, precision=1)
        return b

    b = solver(None)
    first, second = run(b), run(b)
    b.set_schedule(other)
    third = run(b)
    want = run(solver(other))
    for i in range(3):
        assert torch.equal(first[i], second[i]) and not torch.equal(first[i], want[i])
        assert torch.equal(third[i], want[i])
