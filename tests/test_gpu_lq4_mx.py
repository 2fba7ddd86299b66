"""The 4-state FP64 rollouts on the matrix cores (16 scenarios per wave, draws loaded two steps at
a time in groups of 16 steps) at the edges of their layout, against the FP64 oracle: scenario
counts around one wave and one workgroup, horizons around a group and odd, both disturbance
injections, streamed and regenerated draws.  Tolerance: 1e-11 on margins of order one, the bound
of the one-lane FP64 rollouts (a few thousand roundings of 2^-53)."""
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


@pytest.mark.parametrize("inject", [W.INJECT_ODE, W.INJECT_POST])
@pytest.mark.parametrize("N,H", [(1, 1), (15, 16), (16, 17), (17, 31), (63, 32), (65, 33),
                                 (257, 64), (130, 203)])
def test_fp64_margins(R, oracle_mod, N, H, inject):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.01, eps=W.LQ4_EPS, inject=inject,
                      w_half=0.05 if inject == W.INJECT_ODE else 5e-4)
    o = oracle_mod.Oracle(p)
    x = np.array([0.03, -0.02, 0.05, 0.01])
    kap = [0.0, 0.31, 1.0]
    got = {}
    for rng in (R.RNG_STREAM, R.RNG_INLINE):
        g = R.Governor(p, precision=R.PREC_F64, rng_mode=rng)
        got[rng] = g.margin(x, 1.3, -0.4, kap, per_scenario=True)
        assert g.step(x, 1.3, -0.4)["kappa"] == o.bisect(x, 1.3, -0.4, 0, 12)["kappa"]
    for i, k in enumerate(kap):
        worst, per, _, _ = o.candidate(x, o.candidate_v(k, 1.3, -0.4), 0)
        m = got[R.RNG_STREAM]
        assert abs(m["margins"][i] - worst) <= 1e-11
        assert np.array_equal(m["per_scenario"][i], np.asarray(per).astype(np.float32)) or \
            np.max(np.abs(m["per_scenario"][i] - per)) <= 2.0 ** -24 * np.max(np.abs(per))
    a, b = got[R.RNG_STREAM], got[R.RNG_INLINE]
    for key in ("margins", "per_scenario", "per_scenario_j"):
        assert np.array_equal(a[key], b[key])


@pytest.mark.parametrize("N", [1, 16, 70, 300])
@pytest.mark.parametrize("rng_mode", [0, 1])
def test_fp32_rechecks(R, oracle_mod, N, rng_mode):
    # a band wider than every margin: each scenario's verdict comes from the FP64 re-simulation
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=90, dt=0.01, eps=W.LQ4_EPS)
    o = oracle_mod.Oracle(p)
    x = np.array([0.03, -0.02, 0.05, 0.01])
    for q in (0, N // 4):
        g = R.Governor(p, band=3.0, rng_mode=rng_mode, chance_q=q)
        for t, (r, v) in enumerate([(1.6, 0.2), (-1.9, -0.1), (0.2, 0.1)]):
            ref = o.bisect(x, r, v, t, 12) if q == 0 else o.bisect_q(x, r, v, t, 12, q)
            assert g.step(x, r, v)["kappa"] == ref["kappa"], (q, t)
