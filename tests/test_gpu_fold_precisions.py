"""A batch whose instances iterate in both precisions at once: each instance's passes
leave the records of the others alone, so that an instance's results do not depend on
the precision that its neighbours have reached."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def _lp(seed, m, n):
    return lpgen.planted_lp(np.random.default_rng(seed), m=m, n=n, per_col=min(m, 4), name="fold")


@pytest.mark.parametrize("layout", ["rows", "bands"])
def test_results_do_not_depend_on_the_neighbours_precision(layout):
    hard, hard2, easy = _lp(1, 400, 900), _lp(2, 400, 900), _lp(3, 4, 30)
    sols = []
    for other in (hard2, easy):
        b = P.Batch([P.Problem.from_instance(i) for i in (hard, other)])
        b.set_layout(layout)
        # tolerances that nothing reaches: the easy one goes on in FP64, the hard one stays in FP32
        sols.append(b.solve(precision="mixed", rel_tol=1e-300, abs_tol=1e-300, polish_switch_tol=1e-5, stall_checks=0,
                            max_iter=768, check_every=64))
    assert sols[1][1].info["fp64_iters"] > 0 and sols[1][0].info["fp64_iters"] == 0, [s.info for s in sols[1]]
    a, b = sols[0][0], sols[1][0]
    for key in ("iters", "accepted_iters", "checks", "restarts", "exit_code"):
        assert a.info[key] == b.info[key], (key, a.info, b.info)
    assert np.array_equal(a.x, b.x) and np.array_equal(a.y, b.y)
