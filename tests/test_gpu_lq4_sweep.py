"""FP32 set-point sweeps of the 4-state plant with one scenario per lane on the matrix cores:
ragged scenario counts, short last candidate groups, horizons around a group of prefetched draws,
both injections and draw modes, against the FP64 oracle (1e-5 relative, the bound of every FP32
margin) and the quad layout's bookkeeping."""
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
@pytest.mark.parametrize("rng_mode", [0, 1])
# large enough for the one-lane layout, with one, two and three candidates per lane
@pytest.mark.parametrize("N,M,H", [(1985, 127, 1), (2048, 127, 9), (4033, 65, 8), (16385, 16, 17),
                                   (33000, 11, 7), (65000, 33, 3)])
def test_sweep(R, oracle_mod, N, M, H, rng_mode, inject):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.02, eps=W.LQ4_EPS, inject=inject,
                      w_half=0.05 if inject == W.INJECT_ODE else 1e-3)
    o = oracle_mod.Oracle(p, nthreads=8)
    x = np.array([0.05, -0.1, 0.08, 0.02])
    kap = np.linspace(0.0, 1.0, M)
    g = R.Governor(p, rng_mode=rng_mode)
    got = g.margin(x, 1.2, -0.5, kap, per_scenario=True)
    one = R.Governor(p, rng_mode=rng_mode, lanes=1).margin(x, 1.2, -0.5, kap)
    assert np.max(np.abs(got["margins"] - one["margins"])) <= 1e-5
    for i in (0, M // 2, M - 2, M - 1):
        worst, per, _, _ = o.candidate(x, o.candidate_v(float(kap[i]), 1.2, -0.5), 0)
        assert np.max(np.abs(got["per_scenario"][i] - per)) <= 1e-5
        assert abs(got["margins"][i] - worst) <= 1e-5
        assert 0 <= got["per_scenario_j"][i].min() and got["per_scenario_j"][i].max() <= H
