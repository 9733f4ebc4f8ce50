"""The multisection passes of a restart check cut row ranges with cone blocks
finer than the trial passes (one block per range instead of two), and leave one
record per range: as many records as there are cone blocks, whatever the number
of trial ranges is.  Solves that run checks on many cone blocks, before and after
their buffers are made anew, return the same bits."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def test_checks_with_many_cone_blocks_after_a_rebuild():
    inst = lpgen.exp_instance(1, m_zero=300, n=2500, m_nonneg=200, n_exp=420, n_dexp=330)
    p = P.Problem.from_instance(inst)
    first = p.solve(max_iter=192)
    assert first.info["checks"] == 3
    for _ in range(3):  # the same schedule, its device buffers allocated again
        p.set_band_schedule()
        again = p.solve(max_iter=192)
        assert again.info["checks"] == 3 and again.info["restarts"] == first.info["restarts"]
        assert np.array_equal(again.x, first.x) and np.array_equal(again.y, first.y)
