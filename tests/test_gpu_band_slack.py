"""The dual-slack epilogue at the end of the band tiles of G^T: tile counts around a
tile, below and past the records that the trials' passes fold, a batch of unlike
instances; against row blocks, whose sums have another order."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def _lp(m, n):
    return lpgen.planted_lp(np.random.default_rng(n), m=m, n=n, per_col=min(m, 3), name="slack")


def _compare(a, b, precision):
    for key in ("iters", "checks", "exit_code") + (("accepted_iters", "restarts") if precision == "fp64" else ()):
        assert a.info[key] == b.info[key], (key, a.info, b.info)
    # 24 trials and one check: rounding grows by the step's condition, at most 1e4 here
    tol = 1e4 * (2.0**-53 if precision == "fp64" else 2.0**-24)
    for u, v in ((a.x, b.x), (a.y, b.y), (a.lam, b.lam)):
        assert np.max(np.abs(u - v)) <= tol * (1.0 + np.max(np.abs(v))), float(np.max(np.abs(u - v)))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("m,n", [(1, 2), (300, 255), (40, 257), (9000, 120000), (9000, 140000)])
def test_band_tiles_with_the_slack_epilogue_equal_row_blocks(m, n, precision):
    inst = _lp(m, n)
    sols = []
    for layout in ("bands", "rows"):
        prob = P.Problem.from_instance(inst)
        prob.set_layout(layout)
        sols.append(prob.solve(precision=precision, max_iter=24, check_every=24))
    _compare(*sols, precision)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_a_batch_of_unlike_instances(precision):
    insts = [_lp(m, n) for m, n in ((5, 9), (700, 1500), (1, 3), (4000, 9000))]
    sols = []
    for layout in ("bands", "rows"):
        b = P.Batch([P.Problem.from_instance(i) for i in insts])
        b.set_layout(layout)
        sols.append(b.solve(precision=precision, max_iter=24, check_every=24))
    for a, b in zip(*sols):
        _compare(a, b, precision)
