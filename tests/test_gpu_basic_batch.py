"""The basic scheme in batches of many blocks, whose steps are tested by a
launch of their own (one image's steps, and a batch's once few problems are
left, are tested by the next step's inverse pass): every problem of a batch
that crosses the line as its problems finish equals its single solve bit for
bit, on the block passes and the 2-D and 3-D wave passes."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# blocks of the axis-0 passes per problem: 201, 27 (fourteen columns each) and 54; the line is at 8192
@pytest.mark.parametrize("shape,n", [((30, 400), 48), ((81, 729), 310), ((27, 27, 27), 180)],
                         ids=["30x400", "81x729", "27x27x27"])
def test_batch_equals_single(shape, n):
    from paper_1004_1122_amd import lshom
    d = len(shape)
    rng = np.random.default_rng(sum(shape))
    probs = []
    for i in range(n):
        rho = 2.0 + 8.0 * (i % 7) / 6.0
        probs.append(dict(phase=(rng.random(shape) < 0.4).astype(np.uint8), cond=[1.0, rho], E=(1.0, 0.3, -0.4)[:d],
                          tol=1e-5, want_field=True))
    b = lshom.BatchSolver()
    b.prepare(probs, precision=0)
    fields, leff, infos = b.run(method=lshom.METHOD_FFTH, graph_block=4)
    its = [info["iterations"] for info in infos]
    assert max(its) > 2 * min(its), its
    for i in (0, 1, 2, 3, 4, 5, 6, n - 1):
        p = probs[i]
        e, l1, info = lshom.Solver(p["phase"], p["cond"]).solve(p["E"], tol=p["tol"], method=lshom.METHOD_FFTH)
        assert info["iterations"] == its[i] and infos[i]["status"] == 0
        assert info["rel_res"] == infos[i]["rel_res"]
        assert torch.equal(fields[i], e) and np.array_equal(leff[i][:d], l1)
    # stopped by the iteration limit in the middle of a block
    _, _, infos = b.run(method=lshom.METHOD_FFTH, graph_block=4, max_iter=6, allow_fail=True)
    assert all(info["iterations"] == min(6, k) for info, k in zip(infos, its))
    assert all((info["status"] == 0) == (k <= 6) for info, k in zip(infos, its))
