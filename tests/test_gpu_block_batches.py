"""Batches on a grid that runs the block passes (72 x 75: too large for one
block per image, no wave lengths), in both precisions: launches that shrink to
the unfinished problems, the tail's own schedule, the caller's launch shapes
and radices, captured blocks of four iterations over cells and warm starts.
Smaller images run whole FP64 solves in one launch and would pass these without
using any of it."""

import numpy as np
import pytest

from oracle import lshom_oracle as o
from paper_1004_1122_amd import microstructure as ms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPE = (72, 75)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _phase(seed):
    m = ms.grf_two_phase(75, 0.15, 0.4, 10.0, seed=seed)
    return np.ascontiguousarray(m.phase[:SHAPE[0], :SHAPE[1]])


def _problems(rhos, tol=1e-9, seed=0):
    return [dict(phase=_phase(700 + seed + i), cond=[1.0, float(rho)], E=(1.0, 0.5) if i % 2 else (0.0, 1.0), tol=tol,
                 want_field=True) for i, rho in enumerate(rhos)]


def _run(b, **kw):
    fields, leff, infos = b.run(**kw)
    return [f.clone() for f in fields], leff.copy(), infos


@pytest.mark.parametrize("precision", [0, 1])
def test_launches_shrink_to_the_unfinished(precision):
    from paper_1004_1122_amd import lshom
    probs = _problems(np.geomspace(2.0, 5e3, 8), tol=1e-8)
    b = lshom.BatchSolver()
    b.prepare(probs, precision=1)
    for _ in range(2):  # captures, then replays
        fields, leff, infos = _run(b, precision=precision, graph_block=4)
        its = [info["iterations"] for info in infos]
        assert max(its) > 4 * min(its), its
        for i, p in enumerate(probs):
            e, l1, info = lshom.Solver(p["phase"], p["cond"]).solve(p["E"], tol=p["tol"], precision=precision,
                                                                    graph_block=4)
            assert infos[i]["status"] == 0 and its[i] == info["iterations"], i
            assert torch.equal(fields[i], e) and np.array_equal(leff[i][:2], l1), i


@pytest.mark.parametrize("precision", [0, 1])
def test_tail_takes_its_own_schedule(precision):
    """A tail schedule with other radices leaves the problems that finish
    before the tail as they were, bit for bit, and changes the rounding of the
    last ones only."""
    from paper_1004_1122_amd import lshom
    probs = _problems([2.0, 3.0, 4.0, 5.0, 800.0, 900.0], tol=1e-8, seed=50)
    s = lshom.Solver(probs[0]["phase"], probs[0]["cond"])
    base = s.get_schedule(precision)

    def run(tail):
        b = lshom.BatchSolver()
        if tail:
            b.set_schedule(dict(base, radix=[r[::-1] for r in base["radix"]], rows_per_block=2, threads_row=128,
                                tail_rows=2))
        b.prepare(probs, precision=1)
        return _run(b, precision=precision, graph_block=4)

    plain, _, inf0 = run(False)
    tailed, _, inf1 = run(True)
    tol = 1e-9 if precision == 0 else 1e-6
    for i in range(6):
        if i < 4:
            assert torch.equal(plain[i], tailed[i]) and inf0[i]["iterations"] == inf1[i]["iterations"], i
        else:
            assert not torch.equal(plain[i], tailed[i]), i
            assert _rel(tailed[i].cpu().numpy(), plain[i].cpu().numpy()) < tol, i
            assert inf1[i]["rel_res_true"] <= 1.01e-8


@pytest.mark.parametrize("precision", [0, 1])
def test_schedules_shape_the_launches(precision):
    """Radices, rows and block sizes set by the caller: the field agrees with
    the default schedule's to rounding, and other radices do round otherwise."""
    from paper_1004_1122_amd import lshom
    s = lshom.Solver(_phase(3), [1.0, 10.0])
    good = s.get_schedule(precision)
    e0, _, i0 = s.solve((1.0, 0.0), tol=1e-10, precision=precision)
    bar = 1e-12 if precision == 0 else 1e-8
    for change in (dict(threads_row=256, threads_col=256), dict(threads_row=128, threads_col=128),
                   dict(rows_per_block=6), dict(radix=[r[::-1] for r in good["radix"]])):
        s.set_schedule(dict(good, **change))
        assert {k: s.get_schedule(precision)[k] for k in change} == change
        e1, _, i1 = s.solve((1.0, 0.0), tol=1e-10, precision=precision)
        assert i1["iterations"] == i0["iterations"]
        assert float((e1 - e0).norm() / e0.norm()) < bar
        assert torch.equal(e1, e0) == ("radix" not in change)


@pytest.mark.parametrize("warm", [False, True], ids=["cold", "warm"])
@pytest.mark.parametrize("precision", [0, 1])
def test_captured_blocks_over_cells(precision, warm):
    from paper_1004_1122_amd import lshom
    base = _problems([50.0, 100.0, 150.0], seed=90)
    if warm:
        rng = np.random.default_rng(2)
        for p in base:
            lam = ms.lam_field(p["phase"], p["cond"])
            x0 = o.cg(lam, o.optimal_reference(lam), p["E"], n_iter=6)["e"] + 1e-3 * rng.standard_normal((2,) + SHAPE)
            p["x0"] = torch.from_numpy(x0)
    b = lshom.BatchSolver()
    for cell in (None, (1.0, 3.0), None):
        probs = [dict(p, cell=cell) for p in base]
        b.prepare(probs, precision=1)
        fields, leff, infos = _run(b, precision=precision, graph_block=4)
        for i, p in enumerate(probs):
            s = lshom.Solver(p["phase"], p["cond"], cell=cell)
            e, l1, info = s.solve(p["E"], tol=p["tol"], precision=precision, x0=p.get("x0"), graph_block=4)
            assert infos[i]["warm_start_used"] == info["warm_start_used"]
            if all(q["warm_start_used"] for q in infos) or not any(q["warm_start_used"] for q in infos):
                # (beside warm problems, one that starts from E forms its residual by the general pass)
                assert infos[i]["iterations"] == info["iterations"], (cell, i)
                assert torch.equal(fields[i], e) and np.array_equal(leff[i][:2], l1), (cell, i)
            else:
                assert _rel(fields[i].cpu().numpy(), e.cpu().numpy()) <= 1e-6, (cell, i)
