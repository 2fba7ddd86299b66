"""The device's decision and candidate preparation at the edges of their layouts: one candidate,
one wave's worth, one more, and the most a round holds (two candidates per lane of the deciding
wave; more new set-points than the steady-state cache has entries), against the FP64 oracle."""
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


def _updates():
    rng = np.random.default_rng(3)
    return [(0.02 * rng.standard_normal(4), float(r), float(v)) for r, v in
            [(1.9, 0.1), (-1.7, 0.2), (0.3, 0.1), (1.4, -0.6)]]


@pytest.mark.parametrize("M,refine", [(2, 0), (2, 9), (63, 6), (64, 0), (65, 7), (127, 3)])
def test_grid_rounds(R, oracle_mod, M, refine):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=40, H=60, dt=0.02, eps=W.LQ4_EPS)
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, search=R.SEARCH_GRID, M=M, refine=refine)
    for t, (x, r, v) in enumerate(_updates()):
        ref = o.grid(x, r, v, t, M, refine)
        ref = ref[0] if isinstance(ref, tuple) else ref
        got = g.step(x, r, v)
        assert (got["kappa"], got["bisect_passes"]) == (ref["kappa"], ref["passes"]), (t, got, ref)


@pytest.mark.parametrize("K,depth,predict", [(0, 1, True), (1, 6, False), (6, 6, False),
                                             (13, 6, False), (40, 3, True), (40, 6, True)])
def test_bisection_rounds(R, oracle_mod, K, depth, predict):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=40, H=60, dt=0.02, eps=W.LQ4_EPS)
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, K=K, depth=depth, predict=predict)
    for t, (x, r, v) in enumerate(_updates()):
        ref = o.bisect(x, r, v, t, K)
        got = g.step(x, r, v)
        assert (got["kappa"], got["bisect_passes"]) == (ref["kappa"], ref["passes"]), (t, got, ref)
