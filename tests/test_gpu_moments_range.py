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
