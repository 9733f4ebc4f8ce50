"""What the autotuner may change of a batch's schedule: what the layout depends on."""
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def test_autotune_leaves_what_has_no_effect():
    b = P.Batch([P.Problem.from_instance(lpgen.c0_instance(s)) for s in range(2)])
    b.set_layout("rows")
    b.set_schedule(8, 12345, 512)
    iter_max, block_nnz, vec_per_block = b.autotune(2000.0)
    assert iter_max in (4, 8, 16, 32) and (block_nnz, vec_per_block) == (12345, 512)
    assert b.schedule() == (iter_max, 12345, 512)
