"""The 2-norm pass of the diagonal scaling where a row's or a column's magnitude lies so
far from 1 that its square leaves FP64's range, though that of its scaled entries (about
1 after the Ruiz passes) does not; against NumPy, which scales before it squares."""
import numpy as np
import pytest

import lpgen
from test_gpu_scaling import _scaling

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def _lp(side, size, seed=31):
    m, n = 300, 700
    scale = np.ones(m if side == "row" else n)
    scale[[3, 41]] = size
    return lpgen.planted_lp(np.random.default_rng(seed), m, n, per_col=4, **{side + "_scale": scale})


def _check(s, inst, ruiz):
    longest = max(np.diff(inst.row_ptr).max(), np.bincount(inst.col_idx).max())
    tol = (12 * (ruiz + 1) + longest / 2) * 2.0**-53  # as in test_gpu_scaling.py
    for got, want in zip((s.D1, s.D2), _scaling(inst, ruiz, 1)):
        assert np.max(np.abs(got - want) / want) <= tol


@pytest.mark.parametrize("layout", ["rows", "bands"])
@pytest.mark.parametrize("side", ["row", "col"])
@pytest.mark.parametrize("size", [1e-200, 1e-157, 1e-120, 1e120, 1e157, 1e200])
@pytest.mark.parametrize("ruiz", [3, 10])
def test_rows_and_columns_beyond_the_square_root_of_the_range(ruiz, size, side, layout):
    inst = _lp(side, size)
    p = P.Problem.from_instance(inst)
    p.set_layout(layout)
    _check(p.solve(max_iter=1, ruiz_iters=ruiz, l2_pass=1, with_scaling=True), inst, ruiz)


def test_in_a_batch_on_bands():
    insts = [_lp("row", 1e-157, 32), _lp("col", 1e157, 33), lpgen.c0_instance(3)]
    b = P.Batch([P.Problem.from_instance(i) for i in insts])
    b.set_layout("bands")
    for inst, s in zip(insts, b.solve(max_iter=1, with_scaling=True)):
        _check(s, inst, 10)


@pytest.mark.parametrize("layout", ["rows", "bands", "auto"])
@pytest.mark.parametrize("side", ["row", "col"])
def test_a_sum_of_squares_beyond_the_range_keeps_the_factor(side, layout):
    # no Ruiz pass before: the entries' squares themselves overflow
    p = P.Problem.from_instance(_lp(side, 1e200))
    p.set_layout(layout)
    s = p.solve(max_iter=1, ruiz_iters=0, l2_pass=1, with_scaling=True)
    assert np.all(np.isfinite(s.D1) & (s.D1 > 0)) and np.all(np.isfinite(s.D2) & (s.D2 > 0))
    assert np.all((s.D1 if side == "row" else s.D2)[[3, 41]] == 1.0)
