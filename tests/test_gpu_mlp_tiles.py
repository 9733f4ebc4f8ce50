"""Both output tiles of the MLP products, the one-launch bias step and the
output's denormalization, at the sizes where they can go wrong: sides about 64
and 128, batches about the 32- and 64-row blocks of the column sums, an odd
number of 64-row sums, a loss layer wide enough for the wide tile, inputs whose
rows are no multiple of four.  The layer-by-layer comparison and its bounds are
those of test_gpu_mlp."""
import numpy as np
import pytest

import test_gpu_mlp as base

pytestmark = pytest.mark.gpu

P = base.P
torch = base.torch


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


@pytest.mark.parametrize("dims,batch", [((64, 64, 64), 64), ((65, 63, 129), 65), ((127, 129, 1025), 33), ((130, 128, 63), 32),
                                        ((128, 65, 200), 193), ((64, 64, 33000), 130)])
def test_layers_at_the_tiles_edges(dims, batch):
    base.test_layers_match_oracle_on_gpu_activations(dims, batch)


@pytest.mark.parametrize("dims,batch", [((31, 32, 20), 33), ((64, 64, 33000), 130)])
def test_adam_at_the_tiles_edges(dims, batch):
    base.test_adam_steps_match_textbook_update(dims, batch)


@pytest.mark.parametrize("dims,batch", [((203, 64, 66), 7), ((4000, 32, 131), 70), ((8, 64, 40000), 200)])
def test_normalized_output(dims, batch):
    # the standardized network's output times scale plus mean: one fused
    # multiply-add of FP32 values, and its reference rounds twice
    d_in, w, d_out = dims
    rng = np.random.default_rng(batch)
    u, _, ud, _ = base._data(d_in, d_out, batch, 3)
    net = P.MLP(d_in, w, d_out, seed=6)
    im, isd = rng.standard_normal(d_in).astype(np.float32), rng.uniform(0.5, 2, d_in).astype(np.float32)
    om, osd = rng.standard_normal(d_out).astype(np.float32), rng.uniform(0.5, 2, d_out).astype(np.float32)
    net.set_normalization(im, isd, np.zeros(d_out, np.float32), np.ones(d_out, np.float32))
    plain = net.forward(ud).double().cpu().numpy()
    net.set_normalization(im, isd, om, osd)
    got = net.forward(ud).double().cpu().numpy()
    want = plain * osd + om
    assert np.all(np.abs(got - want) <= 2.0**-22 * (np.abs(plain * osd) + np.abs(om)))
    bf = torch.tensor((u - im) * (np.float32(1) / isd)).bfloat16().float().numpy()
    assert np.array_equal(net.activation("input", batch), bf)
