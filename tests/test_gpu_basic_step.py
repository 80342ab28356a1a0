"""The basic scheme's test of a step inside the next one: iteration limits
inside, at the end of and one past a queued block, and the tolerance met at a
step in the middle of a block, on the block passes and both wave passes,
against the oracle (1e-10 at an equal count, the bar of the other tests)."""

import numpy as np
import pytest

from oracle import lshom_oracle as o
from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(100, 60), (81, 90), (81, 243), (27, 27, 81), (20, 18, 14)],
                         ids=lambda s: "x".join(map(str, s)))
def test_limits_and_tolerance(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1004_1122_amd import lshom
    rng = np.random.default_rng(sum(shape))
    phase = rng.integers(0, 2, size=shape).astype(np.uint8)
    cond = np.array([1.0, 9.0])
    lam = ms.lam_field(phase, cond)
    E = [1.0, 0.5, -0.25][:len(shape)]
    s = lshom.Solver(phase, cond)
    for m in (1, 2, 16, 17, 33):
        e, _, info = s.solve(E, tol=0.0, max_iter=m, method=lshom.METHOD_FFTH, allow_fail=True)
        assert info["iterations"] == m
        assert np.linalg.norm(e.cpu().numpy() - o.ffth(lam, 5.0, E, tol=0.0, max_iter=m)["e"]) <= \
            1e-10 * np.linalg.norm(e.cpu().numpy())
    e, _, info = s.solve(E, tol=1e-4, method=lshom.METHOD_FFTH)
    ref = o.ffth(lam, 5.0, E, tol=0.0, max_iter=info["iterations"])["e"]
    assert np.linalg.norm(e.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
    _, _, short = s.solve(E, tol=1e-4, method=lshom.METHOD_FFTH, max_iter=info["iterations"] - 1, allow_fail=True)
    assert short["iterations"] == info["iterations"] - 1 and short["rel_res"] > 1e-4
