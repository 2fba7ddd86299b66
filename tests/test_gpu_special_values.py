"""Special values in the 9-state plant's output y_1 = c_q0 x_7 / (d_0 + d_1 x_9): a denominator that is
zero gives an infinite output, and its margins (infinite where the constraint is a lower bound,
refused where it is an upper one) are those of IEEE division in every precision and layout, as the
FP64 oracle has them."""
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


@pytest.mark.parametrize("precision,lanes", [(0, 1), (0, 16), (1, 0)])
@pytest.mark.parametrize("sign", [-1.0, 1.0])
def test_zero_denominator(R, oracle_mod, sign, precision, lanes):
    p = W.fc9_problem(N=20, H=6)
    c = p.coeffs.copy()
    c[112] = c[113] = 0.0
    # four rows on y_1 alone leave no padding row, whose 0 * inf would be NaN; the other outputs'
    # zero factors multiply finite values
    p = p.replace(coeffs=c, F=np.tile([sign, 0.0, 0.0], (4, 1)), g=np.array([-2.35, 1.0, 2.0, 3.0]))
    o = oracle_mod.Oracle(p)
    x = c[81:90].copy()
    ref, per, _, _ = o.candidate(x, o.candidate_v(0.5, 1.9, 0.5), 0)
    assert ref == -sign * np.inf
    g = R.Governor(p, precision=precision, lanes=lanes)
    m = g.margin(x, 1.9, 0.5, [0.5], per_scenario=True)
    assert m["margins"][0] == ref and np.array_equal(m["per_scenario"][0], np.asarray(per))
    assert g.step(x, 1.9, 0.5)["kappa"] == o.bisect(x, 1.9, 0.5, 0, 12)["kappa"]


def _diverging(N, H, unstable, quad):
    """A fourth state that no output sees and nothing moves but itself: x' = unstable x + quad x^2."""
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.02, eps=0.0, ss_check=0)
    c = p.coeffs.copy()
    c[:16] = np.diag([-1.0, -2.0, -3.0, unstable]).ravel()
    c[19] = c[42] = c[43] = 0.0
    c[20:36] = 0.0
    c[35] = quad
    c[44:52] = [1, 0, 0, 0, 0, 1, 0, 0]
    return p.replace(coeffs=c)


@pytest.mark.parametrize("N,H", [(1, 100), (40, 100), (300, 109)])
def test_fp64_state_that_leaves_the_range(R, oracle_mod, N, H):
    # margins are finite up to the step at which the state overflows; that step is the minimiser
    p = _diverging(N, H, 4.0, 3.0)
    o = oracle_mod.Oracle(p)
    x = np.array([0.05, -0.1, 0.08, 0.02])
    g = R.Governor(p, precision=1)
    m = g.margin(x, 0.3, 0.1, [0.0, 1.0], per_scenario=True)
    assert np.all(m["margins"] == -np.inf) and np.all(m["per_scenario"] == -np.inf)
    for k in range(0, N, max(1, N // 7)):
        j = o.rollout_tangent(x, 0.3, 0, k)[3]
        assert 0 < j < H and m["per_scenario_j"][1, k] == j
    assert g.step(x, 0.3, 0.1)["kappa"] == o.bisect(x, 0.3, 0.1, 0, 12)["kappa"] == 0.0


def test_fp64_state_that_stays_in_range(R, oracle_mod):
    p = _diverging(40, 60, 20.0, 0.0)
    o = oracle_mod.Oracle(p)
    x = np.array([0.05, -0.1, 0.08, 0.02])
    m = R.Governor(p, precision=1).margin(x, 0.3, 0.1, [1.0], per_scenario=True)
    worst, per, _, _ = o.candidate(x, 0.3, 0)
    assert np.isfinite(worst) and abs(m["margins"][0] - worst) <= 1e-11
