"""The 2-D passes along axes of 81, 243 and 729 nodes: each length in each axis
position beside axes the block passes keep (odd, even, tiny), against the
oracle at the bars of the other solver tests (apply 1e-13, CG and the basic
scheme 1e-10 at an equal iteration count, mixed solves against the converged
field), the equilibrium sums, and a batch against single solves."""

import numpy as np
import pytest

from oracle import lshom_oracle as o
from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(81, 81), (81, 63), (63, 81), (243, 10), (10, 243), (243, 16), (81, 243), (729, 6), (6, 729), (3, 729),
          (729, 81)]
ids = ["x".join(map(str, s)) for s in SHAPES]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _problem(shape, n_phases=3):
    rng = np.random.default_rng(sum(shape) + shape[0])
    return rng.integers(0, n_phases, size=shape).astype(np.uint8), rng.uniform(1.0, 30.0, size=n_phases)


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_apply(shape):
    from paper_1004_1122_amd import lshom
    phase, cond = _problem(shape)
    s = lshom.Solver(phase, cond)
    l0 = 0.41 * float(cond.max() + cond.min())
    s.set_reference(l0)
    p = np.random.default_rng(3).standard_normal((2,) + shape)
    q = s.apply(torch.from_numpy(p)).cpu().numpy()
    assert _rel(q, o.apply_A(p, ms.lam_field(phase, cond), l0)) <= 1e-13


@pytest.mark.parametrize("method", ["cg", "basic", "mixed"])
@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_solve(shape, method):
    from paper_1004_1122_amd import lshom
    phase, cond = _problem(shape)
    lam = ms.lam_field(phase, cond)
    l0 = 0.5 * float(cond.max() + cond.min())
    E = [0.8, -0.6]
    s = lshom.Solver(phase, cond)
    if method == "mixed":
        e, leff, info = s.solve(E, tol=1e-8, precision=1)
        ref = o.cg(lam, l0, E, tol=1e-12)["e"]
        assert info["rel_res_true"] <= 1e-8
        assert _rel(e.cpu().numpy(), ref) <= 1e-6
    elif method == "basic":
        e, leff, info = s.solve(E, tol=1e-6, method=lshom.METHOD_FFTH)
        ref = o.ffth(lam, l0, E, tol=0.0, max_iter=info["iterations"])["e"]
        assert _rel(e.cpu().numpy(), ref) <= 1e-10
    else:
        e, leff, info = s.solve(E, tol=1e-9)
        ref = o.cg(lam, l0, E, n_iter=info["iterations"])["e"]
        assert _rel(e.cpu().numpy(), ref) <= 1e-10
    np.testing.assert_allclose(leff, o.leff(lam, e.cpu().numpy()), rtol=1e-10)


@pytest.mark.parametrize("shape", [(81, 243), (63, 81), (243, 27)], ids=lambda s: "x".join(map(str, s)))
def test_equilibrium_history(shape):
    """eta_e of every iterate: the |xi|^2-weighted sums and the cell sums at
    k = 0 of these passes, with and without the history the same iterates."""
    from paper_1004_1122_amd import lshom
    phase, cond = _problem(shape)
    lam = ms.lam_field(phase, cond)
    l0 = 0.5 * float(cond.max() + cond.min())
    s = lshom.Solver(phase, cond)
    e, _, info = s.solve([1.0, 0.0], tol=1e-8, history=64)
    e2, _, info2 = s.solve([1.0, 0.0], tol=1e-8)
    assert info2["iterations"] == info["iterations"] and torch.equal(e, e2)
    for m in (0, 3, info["iterations"]):
        it = o.cg(lam, l0, [1.0, 0.0], n_iter=m)["e"]
        want = o.eta_e(lam, it)
        assert abs(info["history"][m, 1] - want) <= 1e-8 * info["history"][0, 1] + 1e-8 * want


def test_batch_equals_single():
    from paper_1004_1122_amd import lshom
    probs = []
    for i, n in enumerate((81, 243, 81, 243, 81)):
        m = ms.grf_two_phase(n, 0.12, 0.4, 20.0, seed=40 + i)
        probs.append(dict(phase=m.phase, cond=[1.0, 20.0 + i], E=(1.0, 0.3), tol=1e-8, want_field=True))
    for precision in (0, 1):
        b = lshom.BatchSolver()
        b.prepare(probs, precision=1)
        fields, leff, _ = b.run(precision=precision)
        for i, p in enumerate(probs):
            e, l1, _ = lshom.Solver(p["phase"], p["cond"]).solve(p["E"], tol=p["tol"], precision=precision)
            assert torch.equal(fields[i], e) and np.array_equal(leff[i][:2], l1)
