"""Problems that fit in LDS run what lies between a check's products in one workgroup
(bounds open on either side: both rays; rows and columns of several blocks); row
blocks run it in launches of many, with the trials' sums in another order."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("m,n,open_bounds", [(1, 2, False), (60, 150, True), (220, 550, False), (300, 520, True)])
def test_one_workgroup_checks_equal_row_block_checks(m, n, open_bounds, precision):
    inst = lpgen.planted_lp(np.random.default_rng(m), m=m, n=n, per_col=min(m, 4), name="wg")
    if open_bounds:
        inst.l = np.where(np.arange(n) % 7 == 0, -np.inf, inst.l)
        inst.u = np.where(np.arange(n) % 5 == 0, np.inf, inst.u)
    sols = []
    for layout in ("workgroup", "rows"):
        prob = P.Problem.from_instance(inst)
        prob.set_layout(layout)
        sols.append(prob.solve(precision=precision, max_iter=32, check_every=32))
    a, b = sols
    for key in ("iters", "checks", "exit_code") + (("accepted_iters", "restarts") if precision == "fp64" else ()):
        assert a.info[key] == b.info[key], (key, a.info, b.info)
    # 32 trials and one check: rounding grows by the step's condition, at most 1e4 here
    tol = 1e4 * (2.0**-53 if precision == "fp64" else 2.0**-24)
    for u, v in ((a.x, b.x), (a.y, b.y), (a.lam, b.lam)):
        assert np.max(np.abs(u - v)) <= tol * (1.0 + np.max(np.abs(v))), float(np.max(np.abs(u - v)))
