"""Batches with streamed and with regenerated draws (rg_scenarios.rng_mode of the descriptors): both
plants, both injections and, for the 9-state plant, both rollout layouts in every mode reach the
oracle's kappa, agree with each other, and may be mixed in one batch."""
import numpy as np
import pytest

from paper_2510_08288_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_08288_amd import rg
    rg.load_library()
    return rg


def _instances(oracle_mod):
    probs, xs, rs, vps = [], [], [], []
    # 9-state horizons far enough apart that the longest run on groups of lanes, the others one lane
    # per scenario
    for i, (kind, N, H, inject) in enumerate([("lq4", 70, 120, 0), ("lq4", 300, 61, 1),
                                              ("fc9", 900, 40, 0), ("fc9", 700, 45, 1),
                                              ("fc9", 100, 700, 0), ("fc9", 65, 600, 1),
                                              ("lq4", 129, 90, 0)]):
        if kind == "lq4":
            p = W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=N, H=H, dt=0.02, eps=W.LQ4_EPS, inject=inject,
                              w_half=1e-3 if inject else 0.05, scen_seed=30 + i, instance=i)
            x, r, v = 0.02 * np.cos(np.arange(4) + i), 1.5 - 0.4 * i, 0.1
        else:
            p = W.fc9_problem(N=N, H=H, dt=0.004, inject=inject, w_half=8e-5 if inject else 0.02,
                              scen_seed=60 + i, instance=i)
            x, r, v = oracle_mod.Oracle(p).steady_margin(0.5)[1], 1.7 + 0.05 * i, 0.5
        probs.append(p)
        xs.append(x)
        rs.append(r)
        vps.append(v)
    return probs, xs, rs, vps


@pytest.mark.parametrize("kw", [dict(), dict(search=1, M=9, refine=4), dict(block=256, predict=True)])
def test_modes_agree_with_the_oracle(R, oracle_mod, kw):
    probs, xs, rs, vps = _instances(oracle_mod)
    n = len(probs)
    mixed = [R.RNG_STREAM, R.RNG_INLINE, R.RNG_INLINE, R.RNG_STREAM, R.RNG_STREAM, R.RNG_INLINE,
             R.RNG_INLINE]
    batches = [R.Batch(probs, rng_mode=m, **kw) for m in (R.RNG_STREAM, R.RNG_INLINE, mixed)]
    for t in range(2):
        outs = [b.step(xs, rs, vps, use_graph=(t == 1)) for b in batches]
        for i, p in enumerate(probs):
            o = oracle_mod.Oracle(p, nthreads=8)
            if kw.get("search"):
                ref = o.grid(xs[i], rs[i], vps[i], t, 9, 4)
            else:
                ref = o.bisect(xs[i], rs[i], vps[i], t, 12)
            for out in outs:
                assert (out["kappa"][i], out["bisect_passes"][i]) == (ref["kappa"], ref["passes"]), (t, i)
    # near-band margins rechecked in FP64 in every mode
    wide = [R.Batch(probs, rng_mode=m, band=3.0) for m in (R.RNG_STREAM, R.RNG_INLINE)]
    for b in wide:
        out = b.step(xs, rs, vps)
        for i, p in enumerate(probs):
            assert out["kappa"][i] == oracle_mod.Oracle(p, nthreads=8).bisect(xs[i], rs[i], vps[i], 0,
                                                                               12)["kappa"], i
    assert n == len(wide[0].problems)


def test_regenerated_draws_take_no_memory(R):
    import torch
    probs = [W.lq4_problem(seed=W.LQ4_PLANT_SEED, N=16384, H=2000, dt=0.005, eps=W.LQ4_EPS,
                           instance=i) for i in range(4)]  # 1 GB of draws
    args = [[np.zeros(4)] * 4, [0.5] * 4, [0.1] * 4]
    used = []
    for mode in (R.RNG_INLINE, R.RNG_STREAM):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        b = R.Batch(probs, rng_mode=mode)
        b.step(*args)
        used.append(before - torch.cuda.mem_get_info()[0])
        b.close()
    assert used[0] < 0.3e9 and used[1] > 1e9, used
