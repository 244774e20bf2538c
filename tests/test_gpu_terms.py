"""The filter's short evaluations against the functions that define them, value by value.

The FP32 filters take the leave probability, the inversion's first term and the
negative-binomial term from short FP64 evaluations where every nearby number rounds to the
same FP32 value; the rejection sampler's candidate comes from an in-range division and root
and a saturating conversion. Filters show a difference in a last bit only where it moves a
draw or an ancestor; here every value is compared.
"""
import numpy as np
import pytest

import paper_2311_12973_amd as G

pytestmark = pytest.mark.gpu
M = 1 << 20


def _same(prec, term, a, b=0.0, c=0.0):
    x, y = (G.term_batch(prec, term, a, b, c, form=f) for f in (0, 1))
    bad = np.flatnonzero(~((x == y) | (np.isnan(x) & np.isnan(y))))
    a, b, c = np.broadcast_arrays(a, b, c)
    assert len(bad) == 0, (len(bad), [(a[i], b[i], c[i], x[i], y[i]) for i in bad[:5]])
    return x


def _f32(x):
    return np.asarray(x, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("prec", [G.PREC_FP32, G.PREC_FP64])
def test_leave_probability(prec):
    """Hazards from subnormal to where the probability is 1, every FP32 value about 16 (the end of
    the short form), log 2 / 2 (of a reduction step) and 2^-24, zero, negative ones and infinity."""
    print("leave", prec, flush=True)
    rng = np.random.default_rng(1)
    near = [np.arange(-2000, 2000) + int(np.float32(x).view(np.int32)) for x in (16.0, 0.34657359, 0.69314718, 2.0**-24)]
    x = np.concatenate([np.exp(rng.uniform(np.log(1e-44), np.log(200.0), M)), rng.uniform(0.0, 17.0, M),
                        np.concatenate(near).astype(np.int32).view(np.float32).astype(np.float64),
                        [0.0, -0.1, -1e30, np.inf, 1e30, np.nan]])
    p = _same(prec, G.TERM_LEAVE, _f32(x))
    assert 0.0 < p[:M].min() and p[:M].max() == 1.0 and p[2 * M + 16000] == 0.0


@pytest.mark.parametrize("hoisted", [0.0, 1.0])
def test_inversion_first_term(hoisted):
    """(1 - p)^n over n p < 10, from p = 1e-12 to 1/2, a third with one to three trials (at n = 1 the
    value is 1 - p, halfway between two FP32 values for one p in four)."""
    print("inversion", hoisted, flush=True)
    rng = np.random.default_rng(2)
    p = _f32(np.exp(rng.uniform(np.log(1e-12), np.log(0.5), M)))
    p[:1000], p[1000:2000] = 0.5, _f32(0.5 - np.arange(1000) * 2.0**-25)
    n = np.floor(1 + np.minimum(9.99 / p, 2.0**24) * rng.random(M))
    n[::3] = rng.integers(1, 4, len(n[::3]))
    keep = n * p < 10
    f = _same(G.PREC_FP32, G.TERM_INVERSION, n[keep], p[keep], hoisted)
    assert keep.mean() > 0.99 and 0.0 < f.min() < 1e-5 and f.max() == 1.0


def test_negative_binomial_term():
    """Dispersions over [2^-30, 2^30] and beyond both ends, means about the dispersion (where the
    larger of the two changes), far from it, and 0; no cases and up to 2^24."""
    print("negative binomial", flush=True)
    rng = np.random.default_rng(3)
    r = np.exp2(rng.uniform(-32, 32, M))
    r[: M // 2] = np.exp(rng.uniform(-3.0, 6.0, M // 2))
    r[:64] = np.repeat([2.0**-30, np.nextafter(2.0**-30, 0), 2.0**30, np.nextafter(2.0**30, 2.0**31)], 16)
    mu = np.floor(np.exp(rng.uniform(0.0, np.log(2.0**24), M)))
    close = slice(M // 8, M // 4)
    mu[close] = np.maximum(1.0, np.round(r[close] + rng.integers(-2, 3, M // 8)))
    r[M // 4: M // 4 + 4096] = mu[M // 4: M // 4 + 4096]  # equal
    y = np.floor(np.exp(rng.uniform(0.0, np.log(2.0**24), M))) - 1.0
    y[::5] = 0.0
    mu[::11] = 0.0
    v = _same(G.PREC_FP32, G.TERM_NB, y, mu, r)
    assert (np.isinf(v) == ((mu == 0) & (y > 0))).all() and (v[(mu == 0) & (y == 0)] == 0).all()


@pytest.mark.parametrize("prec", [G.PREC_FP32, G.PREC_FP64])
@pytest.mark.parametrize("small", [1.35, 28.0])
def test_rejection_candidate(prec, small):
    """Candidates of up to 2^30 trials, half of them from words at the ends of the uniform's range,
    where the proposal's hat is heaviest: inside, below 0, above n and beyond what 32 bits hold."""
    print("candidate", prec, small, flush=True)
    rng = np.random.default_rng(4)
    n = np.floor(np.exp2(rng.uniform(4.33, 30.0, M) if small < 20 else rng.uniform(small, 30.0, M)))
    lo = np.log(10.1 / n)
    p = np.minimum(_f32(np.exp(lo + (np.log(0.5) - lo) * rng.random(M))), 0.5)
    p[: M // 16] = 0.5
    wu = rng.integers(0, 1 << 32, M, dtype=np.uint64)
    wu[::4] >>= rng.integers(0, 32, len(wu[::4])).astype(np.uint64)
    wu[1::4] = (1 << 32) - 1 - (wu[1::4] >> rng.integers(0, 32, len(wu[1::4])).astype(np.uint64))
    c = wu.astype(np.float64) + 2.0**32 * rng.integers(0, 1 << 21, M)
    ok = np.float32(n) * np.float32(p) >= 10
    k = _same(prec, G.TERM_CANDIDATE, n[ok], p[ok], c[ok])
    assert ok.mean() > 0.99 and (k == -1).any() and (k % 1 == 0.5).any() and ((k >= 0) & (k % 1 == 0)).any()
    assert k.max() <= n.max()


def test_term_batch_rejects_bad_arguments():
    for args in ((2, 0, 0), (0, 4, 0), (0, -1, 0), (0, 0, 2)):
        with pytest.raises(G.Smc2Error) as e:
            G.term_batch(args[0], args[1], 1.0, form=args[2])
        assert e.value.code == G.E_ARG
