"""Exponential-cone projections by lanes, where the seed, the side rule of the
root search or a wave's last lanes can go wrong: every sign pattern of v with
zeros, components decades apart, points beside the cone's boundary and far
along its rays, and counts about a wave and a workgroup; against the FP64
oracle and, where v is built from its projection, against that.  A conic solve
with the cone blocks of a range at its cap follows the oracle's trials."""
import itertools

import numpy as np
import pytest

import lpgen
from oracle import pdcs_oracle as O

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2603_15504_amd")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if P.pdcs_device_count() < 1:
        pytest.skip("no GPU visible")


def _signs(rng):
    signs = np.array(list(itertools.product([-1.0, 0.0, 1.0], repeat=3)))
    v = np.repeat(signs, 40, axis=0)
    return v * 10 ** rng.uniform(-2, 2, v.shape), np.exp(rng.uniform(-2, 2, v.shape))


@pytest.mark.parametrize("dual", [False, True])
def test_every_sign_pattern_matches_the_oracle(dual):
    v, f = _signs(np.random.default_rng(31))
    got = P.pdcs_project_cone("exp_dual" if dual else "exp", v, f)
    ref = O.proj_scaled_exp_dual if dual else O.proj_scaled_exp
    for q in range(v.shape[0]):
        want = ref(v[q], f[q])
        assert np.max(np.abs(got[q] - want)) <= 1e-10 * (1 + np.abs(v[q]).max()), (q, v[q], f[q], got[q], want)


@pytest.mark.parametrize("count", [1, 63, 64, 65, 255, 256, 257])
def test_counts_about_a_wave_and_a_workgroup(count):
    # p = s F a(r), v = p - t F^-1 n(r): both over max(1, e^r) and max(1, e^-r)
    rng = np.random.default_rng(count)
    r = rng.uniform(-30, 30, count)
    s, t = 10 ** rng.uniform(-4, 3, count), 10 ** rng.uniform(-4, 3, count)
    f = np.exp(rng.uniform(-2, 2, (count, 3)))
    a = np.stack([r, np.ones(count), np.exp(r)], 1) * np.minimum(1, np.exp(-r))[:, None]
    n = np.stack([-np.ones(count), r - 1, np.exp(-r)], 1) * np.minimum(1, np.exp(r))[:, None]
    p = s[:, None] * f * a
    v = p - t[:, None] * n / f
    got = P.pdcs_project_cone("exp", v, f)
    scale = np.abs(p).max(1, keepdims=True) + np.abs(v).max(1, keepdims=True)
    assert np.all(np.abs(got - p) <= 1e-9 * (1 + scale))


@pytest.mark.parametrize("n_exp,n_dexp", [(15, 0), (16, 1), (17, 16), (32, 1), (0, 33)])
def test_trials_with_ranges_at_their_cap_follow_the_oracle(n_exp, n_dexp):
    inst = lpgen.exp_instance(9, m_zero=40, n=300, m_nonneg=20, n_exp=n_exp, n_dexp=n_dexp)
    inst.soc = (1,) * 5  # the last nonnegative rows as second-order cones of dimension 1
    ref = O.solve(O.lpdata_from_instance(inst), O.Options(max_iter=64, check_every=64), trace=True)
    sol = P.Problem.from_instance(inst).solve(precision="fp64", max_iter=64, check_every=64, trace_trials=64,
                                              keep_state=True)
    assert len(sol.trace) == 64 == len(ref.trace)
    for row, t in zip(sol.trace, ref.trace):
        assert bool(row[6]) == t["accepted"]
        assert row[1] == pytest.approx(t["eta"], rel=1e-9)
        if t["accepted"]:
            assert row[8] == pytest.approx(t["beta"], rel=1e-9, abs=1e-12)
    assert sol.info["exit_code"] == ref.exit_code
    if not ref.checks_log:  # the 64th trial is rejected: no check
        return
    c = ref.checks_log[0]
    assert sol.state["r_cur"] == pytest.approx(c["r"]["cur"], rel=1e-9)
    assert sol.state["rho_cur"] == pytest.approx(c["rho"]["cur"], rel=2e-5)
    assert sol.state["rho_avg"] == pytest.approx(c["rho"]["avg"], rel=2e-5)
