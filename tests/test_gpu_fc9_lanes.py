"""9-state rollouts by groups of 9 lanes at the edges of their layout (seven scenarios per wave,
28 per workgroup, draws loaded four steps ahead): FP64 margins against the oracle, FP32 margins and
minimising steps equal to the one-lane kernel's.  Tolerance: 1e-11 on margins of order one (a few
thousand FP64 roundings, and tanh and square roots within 3 ulp)."""
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
@pytest.mark.parametrize("N,H", [(1, 1), (6, 2), (7, 3), (8, 4), (27, 5), (28, 8), (29, 9), (57, 35)])
def test_layout_edges(R, oracle_mod, N, H, inject):
    p = W.fc9_problem(N=N, H=H, dt=0.01, inject=inject,
                      w_half=0.02 if inject == W.INJECT_ODE else 2e-4)
    o = oracle_mod.Oracle(p)
    kap = [0.0, 0.37, 1.0]
    x = None
    for rng in (R.RNG_STREAM, R.RNG_INLINE):
        f64 = R.Governor(p, precision=R.PREC_F64, rng_mode=rng)
        if x is None:
            x = f64.equilibrium(0.5) * (1.0 + 0.01 * np.sin(np.arange(9)))
        m = f64.margin(x, 1.9, 0.5, kap, per_scenario=True)
        for i, k in enumerate(kap):
            worst, per, _, _ = o.candidate(x, o.candidate_v(k, 1.9, 0.5), 0)
            assert abs(m["margins"][i] - worst) <= 1e-11
            assert np.max(np.abs(m["per_scenario"][i] - per)) <= 2.0 ** -24 * np.max(np.abs(per))
        assert f64.step(x, 1.9, 0.5)["kappa"] == o.bisect(x, 1.9, 0.5, 0, 12)["kappa"]
        one, grp = (R.Governor(p, lanes=n, rng_mode=rng).margin(x, 1.9, 0.5, kap, per_scenario=True)
                    for n in (1, 16))
        for key in ("margins", "per_scenario", "per_scenario_j"):
            assert np.array_equal(one[key], grp[key]), key


@pytest.mark.parametrize("q", [1, 5])
def test_fp64_chance(R, oracle_mod, q):
    p = W.fc9_problem(N=40, H=60, dt=0.01)
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, precision=R.PREC_F64, chance_q=q)
    x = g.equilibrium(0.5)
    for t, r in enumerate([1.9, 2.1, 0.7]):
        assert g.step(x, r, 0.5)["kappa"] == o.bisect_q(x, r, 0.5, t, 12, q)["kappa"]


@pytest.mark.parametrize("inject", [W.INJECT_ODE, W.INJECT_POST])
@pytest.mark.parametrize("N,H,Kc,n", [(1, 1, 50, 1), (6, 2, 1, 6), (8, 5, 2, 7), (9, 30, 7, 8),
                                      (30, 31, 31, 29), (40, 33, 100, 15)])
def test_weighted_gradient(R, oracle_mod, N, H, Kc, n, inject):
    # entry counts around one group, one wave and more; segments of one step, ragged, longer than
    # the horizon.  The ratio falls over such short horizons, so the minimum is not flat.
    # Tolerance: FP32 sweeps, 1e-4 relative to the largest component.
    p = W.fc9_problem(N=N, H=H, dt=0.002, inject=inject,
                      w_half=0.02 if inject == W.INJECT_ODE else 4e-5)
    o = oracle_mod.Oracle(p)
    x0 = o.steady_margin(0.5)[1]
    rng = np.random.default_rng(N)
    up = np.zeros(N, dtype=np.float32)
    idx = rng.choice(N, n, replace=False)
    up[idx] = rng.uniform(0.5, 1.5, size=n).astype(np.float32)
    v = o.candidate_v(0.4, 1.8, 0.5)
    dk, dth = 0.0, np.zeros(20)
    for k in idx:
        _, dv, d, _, _ = o.rollout_tangent(x0, v, 0, int(k))
        dk += float(up[k]) * dv * (1.8 - 0.5)
        dth += float(up[k]) * d
    for rng_mode in (R.RNG_STREAM, R.RNG_INLINE):
        g = R.Governor(p, Kc=Kc, rng_mode=rng_mode)
        for res in (g.grad(x0, 1.8, 0.5, 0.4, upstream=up),
                    dict(zip(("dkappa", "dtheta"), g._weighted_grad(x0, 1.8, 0.5, 0.4, up)))):
            assert abs(res["dkappa"] - dk) <= 1e-4 * max(abs(dk), 1e-6)
            assert np.max(np.abs(res["dtheta"] - dth)) <= 1e-4 * np.max(np.abs(dth))
