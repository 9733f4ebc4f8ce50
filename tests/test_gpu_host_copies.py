"""What reaches the host in pieces or by a launch: parameters at sizes around whole
pieces, and a solve's outputs below and above the size that the solve hands over
itself, against the device's copies."""
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


@pytest.mark.parametrize("d,width", [(7, 8), (2047, 224), (2048, 256), (2500, 256), (6000, 100)])
def test_parameters_come_back_whole(d, width):
    net = P.MLP(d, width, d)
    want = np.random.default_rng(d).standard_normal(net.params.size).astype(np.float32)
    net.params = want
    assert np.array_equal(net.params, want)
    want = -want
    net.params = want
    assert np.array_equal(net.params, want)


@pytest.mark.parametrize("m,n", [(1, 2), (40, 90), (3000, 13000), (6000, 30000)])
def test_outputs_on_the_host_equal_the_device_copies(m, n):
    inst = lpgen.planted_lp(np.random.default_rng(n), m=m, n=n, per_col=min(m, 3), name="out")
    prob = P.Problem.from_instance(inst)
    for trials in (8, 16):  # a second solve does not touch the first one's outputs
        host = prob.solve(max_iter=trials, check_every=8)
        kept = host.x.copy()
        dev = prob.solve(max_iter=trials, check_every=8, device_out=True)
        for a, b in ((host.x, dev.x), (host.y, dev.y), (host.lam, dev.lam)):
            assert np.array_equal(a, b.cpu().numpy())
        assert host.info["pobj"] == dev.info["pobj"] and np.array_equal(host.x, kept)
