"""Instances that are done: they cost their batch no more passes (seven LPs, of which six
are optimal at their start, against all seven running and against one alone; batches of
fewer than eight are never compacted), and the others' results stay what they are."""
import dataclasses
import time

import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def _done(inst):
    return dataclasses.replace(inst, h=np.zeros(inst.m))  # x = 0 is optimal


def _trial_us(insts, precision):
    b = P.Batch([P.Problem.from_instance(i) for i in insts])
    b.set_layout("rows")
    best = {}
    for _ in range(6):
        for k in (64, 576):
            t0 = time.perf_counter()
            sols = b.solve(max_iter=k, check_every=64, precision=precision, rel_tol=1e-300, abs_tol=1e-300, stall_checks=0)
            best[k] = min(best.get(k, 1e9), time.perf_counter() - t0)
    b.close()
    return (best[576] - best[64]) / 512 * 1e6, sols


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_done_instances_cost_no_passes(precision):
    run = lpgen.planted_lp(np.random.default_rng(5), 40000, 80000, per_col=6)
    full, _ = _trial_us([run] * 7, precision)
    mostly, sols = _trial_us([run] + [_done(run)] * 6, precision)
    alone, one = _trial_us([run], precision)
    assert [s.info["exit_code"] for s in sols] == [1] + [0] * 6
    np.testing.assert_array_equal(sols[0].x, one[0].x)
    # a quarter of what six more running instances cost; the operands of one of a trial's
    # passes alone are about a third
    assert mostly <= alone + 0.25 * (full - alone), (alone, mostly, full)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("layout,windows", [("rows", 1), ("bands", 1), ("bands", 2)])
def test_results_do_not_depend_on_done_neighbours(layout, windows, precision):
    rng = np.random.default_rng(7)
    if windows == 2:  # of the dual vector
        run = lpgen.planted_lp(rng, 2**18 + 5, 3000, row_lengths=np.ones(2**18 + 5, np.int64))
    else:
        run = lpgen.planted_lp(rng, 3000, 6000, per_col=4)
    other = lpgen.planted_lp(rng, 900, 2000, per_col=4)
    sols = []
    for neighbour in (other, _done(other)):
        b = P.Batch([P.Problem.from_instance(i) for i in (neighbour, run)])
        b.set_layout(layout)
        sols.append(b.solve(max_iter=192, check_every=64, precision=precision, rel_tol=1e-300, abs_tol=1e-300,
                            stall_checks=0))
        b.close()
    assert sols[0][0].info["exit_code"] == 1 and sols[1][0].info["exit_code"] == 0
    a, b = sols[0][1], sols[1][1]
    for key in ("iters", "accepted_iters", "checks", "restarts", "exit_code"):
        assert a.info[key] == b.info[key], (key, a.info, b.info)
    assert np.array_equal(a.x, b.x) and np.array_equal(a.y, b.y) and np.array_equal(a.lam, b.lam)
