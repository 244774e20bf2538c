"""Workgroup sizes and launch sizes at their limits: the results do not depend on them."""
import numpy as np
import pytest

import paper_2311_12973_amd as G
from paper_2311_12973_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(preset, n, T, seed=5):
    w = dict(W.preset(preset), T=T)
    if preset == "seir":
        w["truth"] = [*w["truth"][:3], 0.01]  # cases from the second day on
    elif preset == "sir_fp64":
        w["fixed"] = [400]
    y = W.simulate(w["model"], w["obs"], w["n_pop"], w["truth"], T, seed, w.get("fixed", ()), min_frac=0)
    theta = np.array(w["truth"]) * np.exp(np.random.default_rng(seed).normal(0, 0.05, (n, w["D"])))
    return w, y, theta


@pytest.mark.parametrize("nx,block", [(3841, 960), (4096, 960), (4033, 192), (4096, 192), (4096, 448), (4096, 704)])
@pytest.mark.parametrize("preset,prec", [("sir_fp64", G.PREC_FP32), ("sir_fp64", G.PREC_FP64), ("seir", G.PREC_FP32),
                                         ("lingauss", G.PREC_FP64)])
def test_workgroup_sizes_that_round_the_particles_beyond_4096(preset, prec, nx, block):
    """4096 particles fill 64 chunk sums. Sizes that round N_x up further (192 to 4224, 960 to
    4800) leave chunks without a particle and without a sum; what lies behind the sums in LDS,
    the constants of the first days, keeps its values, every day's increment with it."""
    w, y, theta = _case(preset, 3, 14)
    if preset != "lingauss":
        assert (y[1:] > 3).all()  # their constants are not zero
    print("beyond 4096", preset, prec, nx, block, flush=True)
    a = G.pf_loglik(w, theta, y, nx, seed=3, k=1, precision=prec, block=block, trace=True)
    b = G.pf_loglik(w, theta, y, nx, seed=3, k=1, precision=prec, block=1024, trace=True)
    assert np.isfinite(b[0]).all()
    for u, v in zip(a, b):
        assert np.array_equal(u, v)


def test_shapes_at_the_end_of_lds_run_for_every_number_of_filters():
    """SEIR scores at N_x = 2150 fit in rows of 2176 particles only: accepted for few and for many
    filters and for a context of several runs, with the same results."""
    w, y, theta = _case("seir", 513, 3)
    want, want_s = G.pf_score(w, theta, y, 2150, 3, 1, block=64)
    for n in (1, 512, 513):
        print("end of LDS", n, flush=True)
        a, s = G.pf_score(w, theta[:n], y, 2150, 3, 1)
        assert np.array_equal(a, want[:n]) and np.array_equal(s, want_s[:n])
    runs = [dict(T=3, nx=2150, seed=i + 1, y=y) for i in range(2)]
    recs = []
    for block in (0, 64):
        s = G.Sampler(w, runs, N=32, K=2, proposal=G.PROP_LANGEVIN, block=block)
        for _ in range(2):
            s.step()
        recs.append([s.records(r) for r in range(2)])
        s.close()
    assert np.array_equal(recs[0], recs[1])


def test_autotuner_times_the_default_size_too():
    """64 SEIR filters of 100 particles run by default on 384 threads, six waves for two chunks of
    particles, a quarter faster than on the 64 or 128 that N_x fills: the autotuner keeps such a size."""
    w, y, _ = _case("seir", 2, 60)
    kw = dict(N=64, K=2)
    runs = [dict(T=60, nx=100, seed=1, y=y)]
    a, b = G.Sampler(w, runs, **kw), G.Sampler(w, runs, tune=1, **kw)
    print("tuned", b.groups(), "default", a.groups(), flush=True)
    assert a.groups()[0]["block"] == 384 and b.groups()[0]["block"] == 384
    for s in (a, b):
        s.step()
    assert np.array_equal(a.records(), b.records())
    a.close()
    b.close()


@pytest.mark.parametrize("block", [64, 128, 192, 448, 1024])
@pytest.mark.parametrize("nx", [60, 130, 700])
@pytest.mark.parametrize("preset", ["sir_fp64", "seir", "seir_learned"])
@pytest.mark.parametrize("prec", [G.PREC_FP32, G.PREC_FP64])
def test_scores_do_not_depend_on_where_the_flows_are_drawn(prec, preset, nx, block):
    """Scores with flows drawn in place, in several passes of a wave and spread over waves, where
    the probability of leaving S is kept beside the flows or, FP64 SEIR, computed again: the bits of
    the pooled launch, which computes it from the counts."""
    w = dict(W.preset(preset), n_pop=4000.0, T=6)
    truth = np.array(w["truth"])
    if preset == "sir_fp64":
        w["fixed"], truth[1] = [120], 0.12
    else:
        truth[1:4] = 0.12, 0.15, 0.025
    y = np.full((6, 1), 12, dtype=np.int32)
    y[0] = 0 if preset != "sir_fp64" else 12  # SEIR: nobody is exposed yet, and no case on the first day
    theta = np.tile(truth, (4, 1)) * np.exp(np.random.default_rng(nx).normal(0, 0.05, (4, w["D"])))
    print("scores", prec, preset, nx, block, flush=True)
    a, sa = G.pf_score(w, theta, y, nx, 9, 2, precision=prec, schedule=G.SCHED_PER_DRAW, block=block)
    b, sb = G.pf_score(w, theta, y, nx, 9, 2, precision=prec, schedule=G.SCHED_POOLED, block=64)
    assert np.isfinite(b).all() and (sb[:, :2] != 0).all()
    assert np.array_equal(a, b) and np.array_equal(sa, sb)
