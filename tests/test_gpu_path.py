"""Search rounds along the bisection path to the predicted root (later rounds of bisection, of a
grid's refinement and of a batch, where more levels are left than one tree takes): kappa and the
number of verdicts are those of sequential bisection whatever the guess, so they are compared for
equality with the FP64 oracle, and with handles whose rounds are trees.  States and references give
roots all over (0, 1), margins bent by the quadratic term (wrong guesses) and long searches whose
last levels lie below binary32's resolution of the margin."""
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


def _updates(n=5):
    rng = np.random.default_rng(17)
    return [(0.03 * rng.standard_normal(4), float(rng.uniform(-2, 2)), float(rng.uniform(-0.5, 0.5)))
            for _ in range(n)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("K,q", [(12, 0), (7, 0), (30, 0), (12, 400)])
def test_bisection(R, oracle_mod, K, q, precision):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=8200, H=50, dt=0.03, eps=W.LQ4_EPS, quad_scale=0.4)
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, K=K, chance_q=q, precision=precision)
    trees = R.Governor(p, K=K, chance_q=q, precision=precision, depth=2)
    for t, (x, r, v) in enumerate(_updates()):
        ref = o.bisect(x, r, v, t, K) if q == 0 else o.bisect_q(x, r, v, t, K, q)
        got, other = g.step(x, r, v), trees.step(x, r, v)
        assert (got["kappa"], got["bisect_passes"]) == (ref["kappa"], ref["passes"]), (t, got, ref)
        assert (other["kappa"], other["bisect_passes"]) == (ref["kappa"], ref["passes"]), t


@pytest.mark.parametrize("M,refine", [(3, 9), (9, 12), (64, 6)])
def test_grid_refinement(R, oracle_mod, M, refine):
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=8200, H=50, dt=0.03, eps=W.LQ4_EPS, quad_scale=0.4)
    o = oracle_mod.Oracle(p)
    g = R.Governor(p, search=R.SEARCH_GRID, M=M, refine=refine)
    for t, (x, r, v) in enumerate(_updates(4)):
        ref = o.grid(x, r, v, t, M, refine)
        ref = ref[0] if isinstance(ref, tuple) else ref
        got = g.step(x, r, v)
        assert (got["kappa"], got["bisect_passes"]) == (ref["kappa"], ref["passes"]), (t, got, ref)


def test_batch(R, oracle_mod):
    probs = [W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=n, H=h, dt=0.03, eps=W.LQ4_EPS, quad_scale=0.4,
                           instance=i)
             for i, (n, h) in enumerate([(1, 40), (33, 50), (64, 61), (500, 47), (1200, 80)])]
    b = R.Batch(probs, K=20)
    for t, (x, r, v) in enumerate(_updates(3)):
        out = b.step([x] * len(probs), [r] * len(probs), [v] * len(probs))
        for i, p in enumerate(probs):
            ref = oracle_mod.Oracle(p).bisect(x, r, v, t, 20)
            assert (out["kappa"][i], out["bisect_passes"][i]) == (ref["kappa"], ref["passes"]), (t, i)


@pytest.mark.parametrize("N,search,M", [(200000, 0, 64), (500000, 0, 64), (500000, 1, 2)])
def test_allocation_free_step_at_its_scratch_limit(R, N, search, M):
    # without prediction a round of one level holds two candidates at most: 8 B x 2 N of the 8 MiB
    p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=3, dt=0.03, eps=W.LQ4_EPS)
    g = R.Governor(p, predict=False, search=search, M=M)
    x, r, v = _updates(1)[0]
    a = g.step_noalloc(x, r, v)
    g.set_step(0)
    assert a["kappa"] == g.step(x, r, v)["kappa"]
