"""One-block solves of more iterations than one launch holds: 63 blocks of
graph_block iterations.  x, r, p and the two residual sums pass from launch to
launch through memory, so a solve split after 63, 126, 189, .. iterations is
the one-launch solve bit for bit, for CG and the basic scheme, single and in a
batch whose problems stop in different launches."""

import numpy as np
import pytest

from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _same(a, b):
    assert torch.equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    keys = ("iterations", "status", "rel_res", "rel_res_true", "eta_r")
    assert [a[2][k] for k in keys] == [b[2][k] for k in keys]


@pytest.mark.parametrize("method,rho", [("cg", 3e4), ("basic", 300.0)])
@pytest.mark.parametrize("shape", [(45, 45), (27, 64), (63, 63)], ids=lambda s: "x".join(map(str, s)))
def test_split_solves_equal_whole_ones(shape, method, rho):
    from paper_1004_1122_amd import lshom
    m = ms.grf_two_phase(64, 0.1, 0.4, rho, seed=9)
    s = lshom.Solver(np.ascontiguousarray(m.phase[:shape[0], :shape[1]]), [1.0, rho])
    kw = dict(method=lshom.METHOD_FFTH) if method == "basic" else {}
    whole = s.solve((1.0, 0.5), tol=1e-8, graph_block=1024, **kw)
    assert whole[2]["iterations"] > 3 * 63
    for graph_block in (1, 2, 16):
        _same(s.solve((1.0, 0.5), tol=1e-8, graph_block=graph_block, **kw), whole)
    # the last iteration is also the last of a launch, the first of the next, the second
    for max_iter in (63, 64, 65, 126, 127, 128):
        kw2 = dict(kw, tol=0.0, max_iter=max_iter, allow_fail=True)
        _same(s.solve((1.0, 0.5), graph_block=1, **kw2), s.solve((1.0, 0.5), **kw2))


def test_split_batch_equals_single():
    from paper_1004_1122_amd import lshom
    probs = []
    for i, rho in enumerate(np.geomspace(2.0, 3e4, 8)):
        m = ms.grf_two_phase(27, 0.15, 0.4, float(rho), seed=700 + i)
        probs.append(dict(phase=m.phase, cond=[1.0, float(rho)], E=(1.0, 0.5), tol=1e-9, want_field=True))
    b = lshom.BatchSolver()
    b.prepare(probs, precision=0)
    fields, leff, infos = b.run(graph_block=1)
    its = [info["iterations"] for info in infos]
    assert min(its) < 63 and max(its) > 3 * 63, its
    for i, p in enumerate(probs):
        e, l1, info = lshom.Solver(p["phase"], p["cond"]).solve(p["E"], tol=p["tol"])
        assert torch.equal(fields[i], e) and np.array_equal(leff[i][:2], l1) and info["iterations"] == its[i]
