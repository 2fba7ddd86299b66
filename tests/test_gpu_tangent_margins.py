"""The tangent rollout's margins and minimising steps are the rollout's own (its state update and
margin rows are the same operations), so rg_tangent and rg_margin agree bit for bit, and rg_grad
differentiates at the step that rg_margin reports."""
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


@pytest.mark.parametrize("rng_mode", [0, 1])
@pytest.mark.parametrize("kind,lanes", [("fc9", 1), ("fc9", 0), ("lq4", 1), ("lq4", 4)])
def test_tangent_margins_are_the_rollouts(R, kind, lanes, rng_mode):
    if kind == "fc9":
        p = W.fc9_problem(N=600, H=300, dt=0.004)
        args = (R.Governor(p).equilibrium(0.5), 1.9, 0.5)
    else:
        p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=600, H=300, dt=0.01, eps=W.LQ4_EPS)
        args = (np.array([0.03, -0.02, 0.05, 0.01]), 1.3, -0.4)
    g = R.Governor(p, lanes=lanes, rng_mode=rng_mode)
    for kappa in (0.0, 0.35, 1.0):
        tan = g.tangent(*args, kappa)
        m = g.margin(*args, [kappa], per_scenario=True)
        assert np.array_equal(tan["m"], m["per_scenario"][0])
        assert np.array_equal(tan["j"], m["per_scenario_j"][0])
        assert tan["M"] == m["margins"][0]
