"""Results of a batch taken to the GPU together: equal to the host copies of
each result, for more instances than one launch takes, for instances without
rows, into the caller's own buffers, and independent of each other."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


@pytest.mark.parametrize("count", [1, 42, 43, 90])
def test_device_results_equal_host_results(count):
    insts = [lpgen.c0_instance(b, m=20 + 7 * b, n=50 + 13 * b, per_col=4) for b in range(count)]
    batch = P.Batch([P.Problem.from_instance(i) for i in insts])
    host = batch.solve(max_iter=20, check_every=20)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        dev = batch.solve(max_iter=20, check_every=20, device_out=True)
    for h, d in zip(host, dev):
        for name in ("x", "y", "lam"):
            assert np.array_equal(getattr(h, name), getattr(d, name).cpu().numpy())
        assert {k: v for k, v in h.info.items() if k != "time_sec"} == {k: v for k, v in d.info.items() if k != "time_sec"}
    dev[0].x.zero_()
    assert np.array_equal(dev[-1].lam.cpu().numpy(), host[-1].lam)


def test_instances_without_rows():
    none = (np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0), np.zeros(0))
    p = P.Problem(0, 3, 0, *none, c=np.array([1.0, -1.0, 0.0]), l=np.zeros(3), u=np.ones(3))
    q = P.Problem.from_instance(lpgen.c0_instance(1))
    host = P.Batch([p, q]).solve(max_iter=20)
    dev = P.Batch([p, q]).solve(max_iter=20, device_out=True)
    for h, d in zip(host, dev):
        for name in ("x", "y", "lam"):
            assert np.array_equal(getattr(h, name), getattr(d, name).cpu().numpy())


def test_null_arguments_are_refused():
    p = P.Problem.from_instance(lpgen.c0_instance(2))
    r = P.pdcs_solve(p.handle, P.pdcs_options_default(max_iter=5))
    try:
        with pytest.raises(P.PdcsError):
            P.pdcs_results_device([r], [0], [0], [0])
    finally:
        P.pdcs_result_destroy(r)
