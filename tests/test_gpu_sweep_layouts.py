"""A candidate's FP32 margins do not depend on what else a set-point sweep asks for: the 4-state
plant's two sweep layouts (a quad of lanes per scenario, one lane per scenario with one or three
candidates) are chosen by the number of candidates and scenarios and must agree bit for bit, in
every draw mode and injection, also where trajectories leave the range of binary32."""
import numpy as np
import pytest

from paper_2510_08288_amd import workloads as W

pytestmark = pytest.mark.gpu

X = np.array([0.05, -0.1, 0.08, 0.02])
KEYS = ("margins", "per_scenario", "per_scenario_j")


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2510_08288_amd import rg
    rg.load_library()
    return rg


@pytest.mark.parametrize("inject", [W.INJECT_ODE, W.INJECT_POST])
@pytest.mark.parametrize("rng_mode", [0, 1])
# sizes at which all M candidates take one lane per scenario, a single one its quad; the second
# launch of 130 (128 + 2) takes quads by itself
@pytest.mark.parametrize("N,M,H", [(1985, 130, 1), (2100, 130, 9), (4033, 65, 50), (16385, 17, 33),
                                   (20000, 11, 17)])
def test_alone_and_together(R, N, M, H, rng_mode, inject):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.02, eps=W.LQ4_EPS, inject=inject,
                      w_half=0.05 if inject == W.INJECT_ODE else 1e-3)
    g = R.Governor(p, rng_mode=rng_mode)
    kap = np.linspace(0.0, 1.0, M)
    got = g.margin(X, 1.2, -0.5, kap, per_scenario=True)
    for i in (0, 1, M // 2, M - 2, M - 1):
        one = g.margin(X, 1.2, -0.5, kap[i:i + 1], per_scenario=True)
        for key in KEYS:
            assert np.array_equal(got[key][i], one[key][0]), (i, key)


@pytest.mark.parametrize("inject", [W.INJECT_ODE, W.INJECT_POST])
def test_streamed_and_regenerated_draws(R, inject):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=300, H=65, dt=0.02, eps=W.LQ4_EPS, inject=inject,
                      w_half=0.05 if inject == W.INJECT_ODE else 1e-3)
    a, b = (R.Governor(p, rng_mode=m).margin(X, 1.2, -0.5, np.linspace(0, 1, 7), per_scenario=True)
            for m in (0, 1))
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), key


def test_trajectories_that_overflow(R):
    # an unstable state that no output sees (margins stay finite until it overflows), and a
    # quadratic one that blows up within the horizon
    for unstable, quad in ((25.0, 0.0), (60.0, 0.0), (4.0, 3.0)):
        p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=16385, H=100, dt=0.02, eps=0.0, ss_check=0)
        c = p.coeffs.copy()
        c[:16] = np.diag([-1.0, -2.0, -3.0, unstable]).ravel()
        c[19] = c[42] = c[43] = 0.0  # neither set-point nor disturbance moves the fourth state
        c[20:36] = 0.0
        c[20 + 15] = quad
        c[44:52] = [1, 0, 0, 0, 0, 1, 0, 0]
        p = p.replace(coeffs=c)
        g = R.Governor(p)
        kap = np.linspace(0.0, 1.0, 17)
        got = g.margin(X, 0.3, 0.1, kap, per_scenario=True)
        assert np.isfinite(got["per_scenario"]).any() == (unstable < 40.0 and quad == 0.0)
        for i in (0, 16):
            one = g.margin(X, 0.3, 0.1, kap[i:i + 1], per_scenario=True)
            for key in KEYS:
                assert np.array_equal(got[key][i], one[key][0]), (unstable, quad, i, key)
