"""Products of the band layout at tile counts below, at and past a round of the
chip, with several windows, with power-law rows (launches whose LDS follows the
tallest tile) and with rows of many extra slots, against the host's FP64 product."""
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


CASES = {
    "one_row": dict(m=1, n=300, per_col=1),
    "below_half_round": dict(m=255 * 256, n=3000, row_lengths=2),
    "half_round": dict(m=255 * 256 + 1, n=3000, row_lengths=2),
    "past_a_round": dict(m=513 * 256, n=1000, row_lengths=1),
    "three_windows": dict(m=40000, n=3 * 2**18 - 7, per_col=1),
    "power_law": dict(m=90000, n=270000, zipf=True),
    "tall_tiles": dict(m=400 * 1024 + 13, n=3000, row_lengths=2),  # tiles of more than 512 rows
    "long_rows": dict(m=700, n=6000, long_rows=(0, 255, 256, 699)),  # rows with up to 63 extra slots
    "one_long_row": dict(m=1, n=5000, long_rows=(0,)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_products_over_tile_counts(name):
    c = dict(CASES[name])
    rng = np.random.default_rng(17)
    if c.pop("zipf", False):
        c["row_lengths"] = lpgen.zipf_row_lengths(rng, c["m"], 1.5, 3000)
    elif "long_rows" in c:
        rows = c.pop("long_rows")
        c["row_lengths"] = np.where(np.isin(np.arange(c["m"]), rows), c["n"] * 4 // 5, 3)
    elif "row_lengths" in c:
        c["row_lengths"] = np.full(c["m"], c["row_lengths"])
    inst = lpgen.planted_lp(rng, name=name, **c)
    p = P.Problem.from_instance(inst)
    p.set_layout("bands")
    for transpose in (False, True):
        A = inst.scipy_csr().T.tocsr() if transpose else inst.scipy_csr()
        x = rng.standard_normal(A.shape[1])
        want, size = A @ x, abs(A) @ abs(x)
        terms = np.diff(A.indptr) + 8  # roundings of a row's sum, of its products and of the inputs' conversion
        for precision, dtype, u in (("fp64", torch.float64, 2.0**-53), ("mixed", torch.float32, 2.0**-24)):
            xd = torch.tensor(x, dtype=dtype, device="cuda")
            out = torch.full((A.shape[0],), float("nan"), dtype=dtype, device="cuda")
            p.spmv(xd.data_ptr(), out.data_ptr(), transpose=transpose, precision=precision,
                   stream=torch.cuda.current_stream().cuda_stream)
            err = np.abs(out.double().cpu().numpy() - want)
            assert np.all(err <= terms * u * size), (name, transpose, precision, float(np.max(err / (size + 1e-300))))
