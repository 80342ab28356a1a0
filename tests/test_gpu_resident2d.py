"""Whole solves of small 2-D images in one block: the edges of the sizes the
kernel takes (even and odd axes, a few rows, long thin images, the largest
it holds and the first it does not), against the oracle at the bars of the
other solver tests (CG and the basic scheme 1e-10 at an equal iteration count,
mixed solves against the converged field); more iterations than one launch
holds; the block passes (which pass timing selects) with a warm start, many
phases and a cell that is not cubic; a batch of more images than CUs against
single solves."""

import numpy as np
import pytest

from oracle import lshom_oracle as o
from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(3, 4), (4, 3), (5, 9), (9, 5), (27, 27), (3, 1152), (1000, 3), (7, 360), (63, 63), (64, 64), (64, 70),
          (64, 72), (70, 63), (45, 96)]
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


@pytest.mark.parametrize("method", ["cg", "basic"])
def test_more_iterations_than_one_launch(method):
    from paper_1004_1122_amd import lshom
    phase = (np.add.outer(np.arange(45), np.arange(21)) % 7 < 3).astype(np.uint8)
    cond = np.array([1.0, 1e4 if method == "basic" else 3.0])
    lam = ms.lam_field(phase, cond)
    l0 = 0.5 * float(cond.max() + cond.min())
    s = lshom.Solver(phase, cond)
    if method == "basic":
        e, _, info = s.solve([1.0, 0.5], tol=0.0, max_iter=1500, method=lshom.METHOD_FFTH, allow_fail=True)
        assert info["iterations"] == 1500
        ref = o.ffth(lam, l0, [1.0, 0.5], tol=0.0, max_iter=1500)["e"]
        assert _rel(e.cpu().numpy(), ref) <= 1e-10
    else:
        for m in (1, 2, 3):
            e, _, info = s.solve([1.0, 0.5], tol=0.0, max_iter=m, allow_fail=True)
            assert info["iterations"] == m
            assert _rel(e.cpu().numpy(), o.cg(lam, l0, [1.0, 0.5], n_iter=m)["e"]) <= 1e-12


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape", [(27, 27), (63, 63), (45, 60), (64, 70)], ids=lambda s: "x".join(map(str, s)))
def test_equals_block_passes(shape, precision):
    from paper_1004_1122_amd import lshom
    phase, cond = _problem(shape, 256)
    s = lshom.Solver(phase, cond, cell=(1.0, 0.7))
    x0, _, _ = s.solve([1.0, 0.2], tol=1e-2)
    kw = dict(tol=1e-9, precision=1) if precision else dict(tol=0.0, max_iter=9, allow_fail=True)
    for start in (None, x0):
        e, leff, info = s.solve([1.0, 0.2], x0=start, **kw)
        s.set_pass_timing(True)
        e2, leff2, info2 = s.solve([1.0, 0.2], x0=start, **kw)
        s.set_pass_timing(False)
        tol = 1e-7 if precision else 1e-11
        assert _rel(e.cpu().numpy(), e2.cpu().numpy()) <= tol
        np.testing.assert_allclose(leff, leff2, rtol=tol, atol=tol)
        if not precision:
            assert info["iterations"] == info2["iterations"] == 9


def test_batch_equals_single():
    from paper_1004_1122_amd import lshom
    probs = []
    for i in range(300):
        m = ms.grf_two_phase((27, 45, 63)[i % 3], 0.12, 0.4, 20.0, seed=40 + i)
        probs.append(dict(phase=m.phase, cond=[1.0, 20.0 + i], E=(1.0, 0.3), tol=1e-8, want_field=True))
    for precision in (0, 1):
        b = lshom.BatchSolver()
        b.prepare(probs, precision=1)
        fields, leff, _ = b.run(precision=precision)
        for i in (0, 1, 2, 100, 299):
            p = probs[i]
            e, l1, _ = lshom.Solver(p["phase"], p["cond"]).solve(p["E"], tol=p["tol"], precision=precision)
            assert torch.equal(fields[i], e) and np.array_equal(leff[i][:2], l1)


def test_converged_at_the_start():
    """A homogeneous image needs no iteration: the field is the load."""
    from paper_1004_1122_amd import lshom
    for shape in ((63, 63), (81, 81), (100, 60), (27, 27, 27), (30, 32, 20)):
        s = lshom.Solver(np.zeros(shape, np.uint8), np.array([2.0, 3.0]))
        E = (1.0, 0.5, 0.25)[:len(shape)]
        for precision in (0, 1):
            e, leff, info = s.solve(E, tol=1e-6, precision=precision)
            assert info["iterations"] == 0
            np.testing.assert_allclose(leff[:len(shape)], 2.0 * np.array(E), rtol=1e-13)
            for t, v in enumerate(E):
                np.testing.assert_allclose(e[t].cpu().numpy(), v, rtol=1e-13)
