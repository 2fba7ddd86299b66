"""Updates whose candidates are all refused at once (the state lies outside Y): a candidate that
died needs no further rollouts, so the waves that start later run none, in the layouts with several
lanes per scenario as well (nine or four times as many waves).  kappa = 0 and the verdict count are
those of the one-lane layout and of sequential bisection."""
import numpy as np
import pytest

from paper_2510_08288_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2510_08288_amd import rg
    rg.load_library()
    return rg


# rounds of many more scenarios than the card runs at once
@pytest.mark.parametrize("precision,lanes", [(0, 16), (1, 0)])
def test_fc9_waves_of_dead_candidates_run_nothing(R, oracle_mod, precision, lanes):
    # just inside the ratio's bound, every scenario crosses it within some steps
    p = W.fc9_problem(N=40000, H=64)
    x, r, v = p.coeffs[81:90].copy(), 1.9, 0.5
    x[8] = 0.98
    got = R.Governor(p, precision=precision, lanes=lanes).step(x, r, v)
    one = R.Governor(p, precision=0, lanes=1).step(x, r, v)
    for q in (got, one):
        assert (q["kappa"], q["v"], q["status"], q["bisect_passes"]) == (0.0, v, 1, 13)
    assert got["candidates"] == one["candidates"]
    assert got["lane_steps"] < 0.7 * one["lane_steps"], (got, one)


@pytest.mark.parametrize("precision,lanes", [(0, 16), (1, 0)])
def test_fc9_state_outside(R, oracle_mod, precision, lanes):
    p = W.fc9_problem(N=3000, H=64)
    x, r, v = p.coeffs[81:90].copy(), 1.9, 0.5  # the ratio starts below its bound
    ref = oracle_mod.Oracle(p.replace(N=40)).bisect(x, r, v, 0, 12)
    got = R.Governor(p, precision=precision, lanes=lanes).step(x, r, v)
    assert (got["kappa"], got["v"], got["status"], got["bisect_passes"]) == (0.0, v, 1, 13)
    assert ref["kappa"] == 0.0 and got["lane_steps"] == 0
    # a NaN output (0 / 0) refuses as well, at the first step every wave runs
    c = p.coeffs.copy()
    c[110] = c[112] = c[113] = 0.0
    got = R.Governor(p.replace(coeffs=c, ss_check=0), precision=precision, lanes=lanes).step(x, r, v)
    assert (got["kappa"], got["status"]) == (0.0, 1)


def test_lq4_waves_of_dead_candidates_run_nothing(R):
    N = 262144
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=64, dt=0.005, eps=W.LQ4_EPS)
    C = p.coeffs[44:52].reshape(2, 4)
    x, r, v = C[0] / (C[0] @ C[0]) * 1.3, 0.3, 0.1  # y_1 = 1.3
    got = R.Governor(p, precision=1).step(x, r, v)
    one = R.Governor(p, precision=0, lanes=1).step(x, r, v)
    for q in (got, one):
        assert (q["kappa"], q["v"], q["status"], q["bisect_passes"]) == (0.0, v, 1, 13)
    # every wave's first group of 16 steps, if none saw the flag
    assert got["lane_steps"] < 0.6 * got["candidates"] * N * 16, got


@pytest.mark.parametrize("q", [3, 400])
def test_chance_verdict(R, oracle_mod, q):
    # candidates that die after q + 1 violations: the count is exact whichever waves still ran
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=5000, H=40, dt=0.03, eps=W.LQ4_EPS)
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, precision=1, chance_q=q)
    for t, (r, v) in enumerate([(1.9, 0.2), (-1.9, -0.1), (0.4, 0.1)]):
        x = np.array([0.03, -0.02, 0.05, 0.01])
        assert g.step(x, r, v)["kappa"] == o.bisect_q(x, r, v, t, 12, q)["kappa"], t
