"""9-state FP32 rollouts away from the built-in plant: strongly coupled plants, where the derivative's
tanh - 1 and the row sums it adds back cancel, and trajectories that leave the range of binary32.

Tolerance of the coupled plants: 1e-5, the bound of every FP32 margin and a tenth of the recheck
band.  (An FP32 emulation of the derivative with tanh itself has the same state error within 7 % up to
row sums |W| of 236, both below 1.3e-6.)"""
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


def _scaled(N, H, dt, w_scale, a_scale):
    p = W.fc9_problem(N=N, H=H, dt=dt, ss_check=0)
    c = p.coeffs.copy()
    c[:81] *= w_scale
    c[90:99] *= a_scale
    return p.replace(coeffs=c)


@pytest.mark.parametrize("lanes", [1, 16])
@pytest.mark.parametrize("w_scale,a_scale,dt", [(1, 1, 0.002), (10, 10, 0.002), (30, 30, 0.001),
                                                (100, 300, 0.0002)])
def test_strongly_coupled_plants(R, w_scale, a_scale, dt, lanes):
    # near the equilibrium of the decoupled plant, tanh of every state about 0, and 2000 steps on
    p = _scaled(200, 2000, dt, w_scale, a_scale)
    x = p.coeffs[81:90] * (1.0 + 0.002 * np.cos(np.arange(9)))
    args = (x, 0.56, 0.55, [0.0, 0.5, 1.0])
    m32 = R.Governor(p, lanes=lanes, band=0.0).margin(*args, per_scenario=True)
    m64 = R.Governor(p, precision=1).margin(*args, per_scenario=True)
    assert np.all(np.isfinite(m64["per_scenario"]))
    assert np.max(np.abs(m32["per_scenario"] - m64["per_scenario"])) <= 1e-5


@pytest.mark.parametrize("inject", [W.INJECT_ODE, W.INJECT_POST])
def test_trajectories_that_overflow(R, oracle_mod, inject):
    # a state with negative decay leaves binary32 (and, over the longer horizon, binary64)
    for H, unstable, finite64 in ((200, 60.0, True), (900, 80.0, False)):
        p = W.fc9_problem(N=60, H=H, dt=0.01, ss_check=0, inject=inject,
                          w_half=0.02 if inject == W.INJECT_ODE else 2e-4)
        c = p.coeffs.copy()
        c[:81] = 0.0
        c[90 + 7] = -unstable  # the eighth state, which no output and no other state sees
        p = p.replace(coeffs=c)
        x = c[81:90].copy()
        args = (x, 0.9, 0.5, [0.0, 0.4, 1.0])
        one, grp = (R.Governor(p, lanes=n).margin(*args, per_scenario=True) for n in (1, 16))
        for key in ("margins", "per_scenario"):
            assert np.array_equal(one[key], grp[key]), key
        assert np.all(one["per_scenario"] == -np.inf)
        m64 = R.Governor(p, precision=1).margin(*args, per_scenario=True)
        o = oracle_mod.Oracle(p)
        for i, k in enumerate(args[3]):
            worst, per, _, _ = o.candidate(x, o.candidate_v(k, 0.9, 0.5), 0)
            assert np.isfinite(worst) == finite64
            assert m64["margins"][i] == worst or abs(m64["margins"][i] - worst) <= 1e-11


@pytest.mark.parametrize("kind,N,H", [("lq4", 33, 80), ("lq4", 500, 203), ("fc9", 20, 60), ("fc9", 301, 150)])
def test_fp64_updates(R, oracle_mod, kind, N, H):
    # kappa, the worst margin of the result and, of single candidates, the minimising steps
    if kind == "lq4":
        p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.01, eps=W.LQ4_EPS)
        x, r, v = np.array([0.03, -0.02, 0.05, 0.01]), 1.3, -0.4
    else:
        p = W.fc9_problem(N=N, H=H, dt=0.01)
        x, r, v = oracle_mod.Oracle(p).steady_margin(0.5)[1] * (1.0 + 0.01 * np.sin(np.arange(9))), 1.9, 0.5
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, precision=1)
    got, ref = g.step(x, r, v), o.bisect(x, r, v, 0, 12)
    assert got["kappa"] == ref["kappa"] and abs(got["worst"] - ref["worst"]) <= 1e-11
    g.set_step(0)
    m = g.margin(x, r, v, [0.4], per_scenario=True)
    vc = o.candidate_v(0.4, r, v)
    for k in range(0, N, max(1, N // 13)):
        mk, _, _, j, _ = o.rollout_tangent(x, vc, 0, k)
        assert m["per_scenario_j"][0, k] == j and abs(m["per_scenario"][0, k] - mk) <= 2.0 ** -23
