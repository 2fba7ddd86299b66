"""The options in force describe a handle's whole launch schedule: a handle created with the depth
another resolved runs the same rounds (the tree beside the predicted round and the rounds along the
predicted path included), so a tuned schedule loses nothing by being written down, and the
autotuners time the schedule that runs by default."""
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


def _lq4(N, H=50, quad=0.0):
    return W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.03, eps=W.LQ4_EPS, quad_scale=quad)


def _updates(n=6):
    rng = np.random.default_rng(17)
    return [(0.03 * rng.standard_normal(4), float(rng.uniform(-2, 2)), float(rng.uniform(-0.5, 0.5)))
            for _ in range(n)]


def _rounds(g, ups=None):
    g.reset()
    g.set_step(0)
    return [(q["rounds"], q["candidates"], q["kappa"]) for q in (g.step(*u) for u in ups or _updates())]


@pytest.mark.parametrize("N,kw", [(64, {}), (8200, {}), (64, dict(precision=1)), (8200, dict(precision=1)),
                                  (200000, {}), (8200, dict(chance_q=5)),
                                  (3000, dict(search=1, M=9, refine=12))])
def test_resolved_depth_runs_the_same_rounds(R, N, kw):
    p = _lq4(N)
    auto = R.Governor(p, **kw)
    explicit = R.Governor(p, depth=auto.options.depth, lanes=auto.options.lanes, **kw)
    assert explicit.options.depth == auto.options.depth
    assert _rounds(auto) == _rounds(explicit)


def test_rounds_along_the_predicted_path(R):
    # linear plant: the margin is affine near the root, so the path through two admitted candidates
    # replaces most of the six rounds that trees of two levels take
    p = _lq4(8200)
    path = R.Governor(p)
    trees = R.Governor(p, predict=False, depth=2)
    a, b = [], []
    for x, r, v in _updates(12):
        for g, out in ((path, a), (trees, b)):
            g.reset()  # every update a handle's first: no previous kappa to follow
            g.set_step(0)
            out.append(g.step(x, r, v))
    assert [q["kappa"] for q in a] == [q["kappa"] for q in b]
    searched = [i for i, q in enumerate(b) if q["rounds"] == 6 and q["kappa"] > 0.25]
    assert len(searched) >= 3
    assert np.mean([a[i]["rounds"] for i in searched]) <= 4.0, [a[i]["rounds"] for i in searched]


def test_path_rounds_stay_within_the_plan(R):
    # margins bent by the quadratic term (wrong guesses): never more rounds than trees alone and one
    # for the predicted round, and one more for a grid's refinement
    p = _lq4(8200, quad=0.4)
    g = R.Governor(p, K=30)
    assert max(r for r, _, _ in _rounds(g)) <= 1 + -(-30 // g.options.depth)
    g = R.Governor(p, search=1, M=9, refine=12)
    assert max(r for r, _, _ in _rounds(g)) <= 2 + -(-12 // g.options.depth)


def test_tuned_handle_keeps_its_path(R):
    p = _lq4(8200)
    r_seq = W.reference_sequence(5, 8, switch_every=2, lo=-2.5, hi=2.5)
    g = R.Governor(p)
    best = g.autotune(np.zeros(4), 0.0, r_seq)
    kw = {k: best[k] for k in ("lanes", "block", "depth", "speculate")}
    again = R.Governor(p, predict=bool(best["predict"]), **kw)
    assert _rounds(g) == _rounds(again)
    plain = R.Governor(p)
    if (best["depth"], best["lanes"], best["predict"]) == (plain.options.depth, plain.options.lanes, 1):
        assert [x[:2] for x in _rounds(g)] == [x[:2] for x in _rounds(plain)]


@pytest.mark.parametrize("count,N", [(3, 64), (6, 500), (20, 2000)])
def test_batches(R, count, N):
    probs = [_lq4(N, H=30 + 5 * i).replace(instance=i) for i in range(count)]
    auto = R.Batch(probs)
    explicit = R.Batch(probs, depth=auto.options.depth)
    assert explicit.options.depth == auto.options.depth
    for x, r, v in _updates(4):
        a, b = (bt.step([x] * count, [r] * count, [v] * count) for bt in (auto, explicit))
        for key in ("rounds", "candidates", "kappa"):
            assert np.array_equal(a[key], b[key]), key
