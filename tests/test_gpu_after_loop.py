"""Margins, gradients and tangents asked of a handle right after a closed loop whose last updates
were decided ahead (their probes ran beside an earlier update's round, from the states those updates
start in): they belong to the state and candidates of the call, as on a fresh handle."""
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


@pytest.mark.parametrize("T,r", [(3, 0.05), (6, 0.05), (6, 3.0), (12, 3.0)])
def test_calls_after_a_closed_loop(R, oracle_mod, T, r):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=256, H=200, dt=0.005, eps=W.LQ4_EPS)
    g = R.Governor(p)
    out = g.closed_loop(np.zeros(4), 0.0, np.full(T, r))
    assert out["rounds"][-1] == 0  # decided ahead
    fresh = R.Governor(p)
    x, kap = np.array([0.02, -0.01, 0.01, 0.0]), np.linspace(0.0, 1.0, 20)
    for h in (g, fresh):
        h.set_step(40)
    a, b = (h.margin(x, 0.7, 0.1, kap, per_scenario=True) for h in (g, fresh))
    for key in ("margins", "per_scenario", "per_scenario_j"):
        assert np.array_equal(a[key], b[key]), key
    ref = oracle_mod.Oracle(p).candidate(x, oracle_mod.Oracle.candidate_v(float(kap[7]), 0.7, 0.1), 40)
    assert abs(a["margins"][7] - ref[0]) <= 1e-5
    for name in ("grad", "tangent"):
        g.closed_loop(np.zeros(4), 0.0, np.full(T, r))
        for h in (g, fresh):
            h.set_step(40)
        a, b = (getattr(h, name)(x, 0.7, 0.1, 0.4) for h in (g, fresh))
        assert (a["M"], a["dkappa"]) == (b["M"], b["dkappa"])
