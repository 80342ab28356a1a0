"""Mixed solves of small 2-D images, whose iterations at high contrast
outnumber the unknowns, so that the rounding of the FP32 steps decides whether
a solve converges: a plain solve takes the steps of the passes, bit for bit
those of a solve with pass timing on, and the 27^2 solves at contrast 1e4 that
the passes bring to 1e-9 still arrive there."""

import numpy as np
import pytest

from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("shape", [(9, 9), (27, 27), (27, 45), (63, 63), (64, 70)], ids=lambda s: "x".join(map(str, s)))
def test_equals_the_timed_passes(shape):
    from paper_1004_1122_amd import lshom
    m = ms.grf_two_phase(max(shape), 0.15, 0.4, 200.0, seed=31)
    s = lshom.Solver(np.ascontiguousarray(m.phase[:shape[0], :shape[1]]), [1.0, 200.0])
    for kw in (dict(), dict(graph_block=4), dict(graph_block=0), dict(refresh_every=7)):
        e, leff, info = s.solve((1.0, 0.5), tol=1e-9, precision=1, **kw)
        s.set_pass_timing(True)
        e2, leff2, info2 = s.solve((1.0, 0.5), tol=1e-9, precision=1, **kw)
        s.set_pass_timing(False)
        assert torch.equal(e, e2) and np.array_equal(leff, leff2), kw
        assert (info["iterations"], info["refreshes"]) == (info2["iterations"], info2["refreshes"]), kw


def test_high_contrast_27():
    from paper_1004_1122_amd import lshom
    for seed in range(700, 708):
        m = ms.grf_two_phase(27, 0.15, 0.4, 1e4, seed=seed)
        s = lshom.Solver(m.phase, [1.0, 1e4])
        for E in ((0.0, 1.0), (1.0, 0.5)):
            _, _, info = s.solve(E, tol=1e-9, precision=1, max_iter=3000, allow_fail=True)
            assert info["status"] == 0 and info["rel_res_true"] <= 1e-9, (seed, E, info)
