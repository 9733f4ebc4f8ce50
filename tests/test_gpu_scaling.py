"""The diagonal scaling (Section 2.6: Ruiz passes, then one pass of square roots of
2-norms) against NumPy, where its kernels can go wrong: rows longer than a row
block, empty rows, blocks of more than 256 rows, several windows, an odd and an
even number of passes, batches; and a batch that leaves the band tiles for row
blocks while it runs (whose scaled CSR values are made at that point)."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def _instance(name):
    rng = np.random.default_rng(23)
    if name == "long_rows":
        lengths = np.array([3000, 0, 1, 2048, 2049, 7, 0] + [3] * 400)
        return lpgen.planted_lp(rng, lengths.size, 4000, row_lengths=lengths)
    if name == "short_rows":  # a block of about two thousand rows of one entry
        return lpgen.planted_lp(rng, 5000, 300, row_lengths=np.ones(5000, np.int64))
    if name == "windows":
        return lpgen.planted_lp(rng, 3000, 2 * 2**18 + 5, per_col=1)
    if name == "lds":  # one workgroup's LDS; rows of up to 64 entries, empty ones, more rows and columns than threads
        lengths = np.array([64, 0, 1, 4, 5, 0] + [2] * 500)
        return lpgen.planted_lp(rng, lengths.size, 600, row_lengths=lengths)
    if name == "lds_tiny":
        return lpgen.planted_lp(rng, 3, 5, per_col=1)
    return lpgen.planted_lp(rng, 700, 1500, per_col=4, row_scale=10.0 ** rng.uniform(-3, 3, 700))


def _scaling(inst, ruiz, l2):
    A = abs(inst.scipy_csr()).tocoo()
    D1, D2 = np.ones(inst.m), np.ones(inst.n)
    for k in range(ruiz + l2):
        e = D1[A.row] * A.data * D2[A.col]
        sr, sc = np.zeros(inst.m), np.zeros(inst.n)
        if k < ruiz:
            np.maximum.at(sr, A.row, e)
            np.maximum.at(sc, A.col, e)
        else:
            np.add.at(sr, A.row, e * e)
            np.add.at(sc, A.col, e * e)
        p = 0.5 if k < ruiz else 0.25
        D1 /= np.where(sr > 0, sr, 1.0) ** p
        D2 /= np.where(sc > 0, sc, 1.0) ** p
    return D1, D2


@pytest.mark.parametrize("layout", ["rows", "bands", "auto"])
@pytest.mark.parametrize("name,ruiz,l2", [("lds", 10, 1), ("lds", 3, 0), ("lds", 0, 0), ("lds_tiny", 10, 1), ("long_rows", 10, 1), ("short_rows", 3, 0), ("windows", 2, 1), ("plain", 10, 1),
                                          ("plain", 0, 1), ("plain", 0, 0)])
def test_scaling_matches_numpy(name, ruiz, l2, layout):
    inst = _instance(name)
    p = P.Problem.from_instance(inst)
    p.set_layout(layout)
    s = p.solve(max_iter=1, ruiz_iters=ruiz, l2_pass=l2, with_scaling=True)
    longest = max(np.diff(inst.row_ptr).max(), np.bincount(inst.col_idx).max())
    tol = (12 * (ruiz + l2) + longest / 2) * 2.0**-53  # 6 roundings a pass, a sum of squares' under a fourth root; twice
    for got, want in zip((s.D1, s.D2), _scaling(inst, ruiz, l2)):
        assert np.max(np.abs(got - want) / want) <= tol


def test_batch_scaling_equals_the_single_problems():
    insts = [_instance("plain"), _instance("long_rows"), lpgen.c0_instance(3)]
    b = P.Batch([P.Problem.from_instance(i) for i in insts])
    for layout in ("rows", "bands"):
        b.set_layout(layout)
        for inst, s in zip(insts, b.solve(max_iter=1, with_scaling=True)):
            p = P.Problem.from_instance(inst)
            p.set_layout(layout)
            one = p.solve(max_iter=1, with_scaling=True)
            np.testing.assert_allclose(s.D1, one.D1, rtol=1e-14)
            np.testing.assert_allclose(s.D2, one.D2, rtol=1e-14)


def test_batch_that_leaves_the_bands_while_running():
    # 16 LPs of 3e5 nonzeros: band tiles until half of them are done, row blocks after
    insts = [lpgen.planted_lp(np.random.default_rng(300 + b), 18000 + 97 * b, 2 * (18000 + 97 * b), per_col=8) for b in range(16)]
    batch = P.Batch([P.Problem.from_instance(i) for i in insts])
    assert batch.band_schedule()["built_rows"] > 0
    sols = batch.solve(rel_tol=3e-3, abs_tol=0.0, max_iter=60000)
    for inst, s in zip(insts, sols):
        assert s.info["status"] == "optimal"
        res = np.max(np.abs(inst.scipy_csr() @ s.x - inst.h))
        assert res <= 3e-3 * 1.001 * (1 + max(np.max(np.abs(inst.h)), np.max(np.abs(inst.scipy_csr() @ s.x))))
    assert len({s.info["iters"] for s in sols}) > 1
