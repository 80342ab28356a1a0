"""The block passes with 128 and with 256 threads per block: the size of a
block follows how far a launch fills the chip, and the sums are formed in one
order either way, so solves agree bit for bit (fields, effective conductivity,
residuals, equilibrium history; CG, basic scheme, pipelined CG, mixed; scalar
and tensor phases; fewer elements than threads up to several per thread)."""

import numpy as np
import pytest

from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(70, 75), (105, 75), (100, 100), (255, 30), (45, 255), (360, 125), (9, 8, 7), (15, 25, 21), (30, 25, 32)]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _solvers(shape, tensor):
    from paper_1004_1122_amd import lshom
    rng = np.random.default_rng(sum(shape))
    phase = rng.integers(0, 3, size=shape).astype(np.uint8)
    cond = rng.uniform(1.0, 20.0, size=3)
    if tensor:
        d = len(shape)
        m = rng.standard_normal((3, d, d))
        cond = np.stack([np.eye(d) * c + 0.2 * (a + a.T) for c, a in zip(cond + 2.0, m)])
    for nt in (0, 128, 256):
        s = lshom.Solver(phase, cond)
        for precision in (0, 1):
            q = s.get_schedule(precision)
            q.update(threads_row=nt, threads_col=nt)
            s.set_schedule(q)
        yield s


@pytest.mark.parametrize("kind", ["cg", "history", "basic", "pipelined", "mixed", "tensor"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_same_bits(shape, kind):
    from paper_1004_1122_amd import lshom
    if kind == "history" and any(n % 2 == 0 for n in shape):
        pytest.skip("the history needs odd axes")
    kw = {"cg": {}, "history": dict(history=64), "basic": dict(method=lshom.METHOD_FFTH, max_iter=2000),
          "pipelined": dict(method=lshom.METHOD_PIPECG), "mixed": dict(precision=1), "tensor": {}}[kind]
    E = (1.0, 0.4, -0.3)[:len(shape)]
    ref = None
    for s in _solvers(shape, kind == "tensor"):
        e, leff, info = s.solve(E, tol=1e-6, **kw)
        got = (e.cpu().numpy(), np.array(leff), info["iterations"], info["rel_res_true"], info.get("history"))
        if ref is None:
            ref = got
            continue
        for a, b in zip(got, ref):
            np.testing.assert_array_equal(a, b)
