"""Walker sums of the moments over the range of displacements a caller can
have, against sums that round once (math.fsum of the same terms)."""
import math

import numpy as np
import pytest

from paper_2308_05007_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2308_05007_amd import binding
    binding.lib()
    return binding


def _displacements(g, n, ref):
    cell, off, img = g.walkers()
    c = np.stack([cell % n[0], (cell // n[0]) % n[1], cell // (n[0] * n[1])]).astype(np.int64)
    return ((c + img.astype(np.int64) * np.asarray(n)[:, None]).astype(float) - np.asarray(ref)[:, None]) + off


def _chain(nw):
    """Error of the sums in double, relative to the sum of the magnitudes: 16
    walkers a thread, 8 folds, the chunks of 4096, and the product's rounding."""
    return (16 + 8 + -(-nw // 4096) + 1) * 2.0 ** -53


@pytest.mark.parametrize("precision", ("fp64", "fp32"))
@pytest.mark.parametrize("nw,ref", ((50_001, (1e3, 2e12, 8.0)), (4097, (-1e13, 8.0, 8.0)), (50_001, (1e12, 8.0, 3e10)),
                                    (1, (8.0, 8.0, 1e150)), (300, (math.inf, 8.0, 8.0)), (300, (8.0, math.nan, 1e3)),
                                    (300, (8.0, 1e200, -math.inf))))
def test_far_references(B, nw, ref, precision):
    n = (18, 15, 21)
    dom = W._domain(n, ("periodic",) * 3, 0.8, (1e-4, 0, 0), 0.1, seed=nw, u0=(0.05, -0.02, 0.01), precision=precision)
    g = B.build_domain(dict(domain=dom, walkers=dict(kind="uniform", n=nw, ref=ref)))
    g.set("sort_every", 4)
    g.step(9)
    with np.errstate(all="ignore"):
        dv = _displacements(g, n, ref)
        terms = np.concatenate([dv, dv * dv])
    for m in (g.moments(), g.moments(noalloc=True), g.moments()):
        for got, t in zip((*m["sum"], *m["sumsq"]), terms):
            if np.isfinite(t).all():
                assert abs(got - math.fsum(t)) <= _chain(nw) * np.abs(t).sum() + np.spacing(abs(got)), (got, t[:4])
            else:
                assert np.array_equal(got, t.sum(), equal_nan=True), (got, t[:4])


# From 2^-11 on every term's 53 bits are held, what remains are the roundings of
# the last combination; below, the sums are in double.
@pytest.mark.parametrize("nw", (1, 1000, 100_003))
@pytest.mark.parametrize("scale", (1e-1, 5e-3, 5e-4, 1e-5, 1e-6, 1e-12, 1e-25))
def test_small_displacements(B, nw, scale):
    n, ref = (18, 15, 21), (0.0, 0.0, 0.0)
    xyz = scale * (0.5 + np.random.default_rng(nw).uniform(size=(nw, 3)))
    dom = W._domain(n, ("periodic",) * 3, 0.8, (0, 0, 0), 0.0, seed=1)
    g = B.build_domain(dict(domain=dom, walkers=dict(kind="explicit", n=nw, xyz=xyz, ref=ref)))
    dv = _displacements(g, n, ref)
    assert np.array_equal(dv, xyz.T)
    for m in (g.moments(), g.moments(noalloc=True)):
        for a in range(3):
            for got, terms in ((m["sum"][a], dv[a]), (m["sumsq"][a], dv[a] * dv[a])):
                want = math.fsum(terms)
                tol = 4 * np.spacing(want) if scale >= 5e-3 else (_chain(nw) * want + np.spacing(want))
                assert abs(got - want) <= tol, (a, got, want)


def test_walkers_on_the_reference(B):
    """All of them, or on two axes, or all but one: sums of zeros are zero."""
    n, nw, ref = (18, 15, 21), 5000, (8.5, 7.25, 3.0)
    dom = W._domain(n, ("periodic",) * 3, 0.8, (0, 0, 0), 0.0, seed=1)
    xyz = np.tile(np.array(ref), (nw, 1))
    for step in (0.0, 0.25, 1e-9):
        xyz[nw // 2, 0] = ref[0] + step
        g = B.build_domain(dict(domain=dom, walkers=dict(kind="explicit", n=nw, xyz=xyz, ref=ref)))
        dx = xyz[nw // 2, 0] - ref[0]
        for m in (g.moments(), g.moments(noalloc=True)):
            assert np.array_equal(m["sum"], [dx, 0.0, 0.0]) and np.array_equal(m["sumsq"], [dx * dx, 0.0, 0.0])
