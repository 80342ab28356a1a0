"""The operator product and BiCG on 3-D grids of 27, 81 and 243 nodes per axis
(the wave passes), against the oracle: apply within 1e-13 and BiCG within
1e-10 of the oracle's iterate, the bars the block passes are held to."""

import numpy as np
import pytest

from oracle import lshom_oracle as o
from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _problem(shape, seed):
    rng = np.random.default_rng(seed)
    phase = rng.integers(0, 3, size=shape).astype(np.uint8)
    return phase, rng.uniform(1.0, 40.0, size=3)


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("shape", [(27, 27, 81), (27, 81, 27), (81, 27, 27), (27, 27, 243), (243, 27, 27)],
                         ids=lambda s: "x".join(map(str, s)))
def test_apply(shape):
    from paper_1004_1122_amd import lshom
    phase, cond = _problem(shape, sum(shape))
    s = lshom.Solver(phase, cond)
    l0 = 0.41 * float(cond.max() + cond.min())
    s.set_reference(l0)
    p = np.random.default_rng(3).standard_normal((3,) + shape)
    q = s.apply(torch.from_numpy(p)).cpu().numpy()
    ref = o.apply_A(p, ms.lam_field(phase, cond), l0)
    assert _rel(q, ref) <= 1e-13


def test_bicg():
    from paper_1004_1122_amd import lshom
    shape = (27, 81, 27)
    phase, cond = _problem(shape, 5)
    s = lshom.Solver(phase, cond)
    E = (0.3, 1.0, -0.2)
    e, _, info = s.solve(E, tol=1e-8, method=lshom.METHOD_BICG)
    l0 = 0.5 * float(cond.max() + cond.min())
    ref = o.bicg(ms.lam_field(phase, cond), l0, list(E), n_iter=info["iterations"])["e"]
    assert _rel(e.cpu().numpy(), ref) <= 1e-10
