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
