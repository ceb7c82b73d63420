"""Moments at the edges of their chunks, against sums that round once: the
walkers' sums are exact up to the last rounding (math.fsum of the same terms),
wherever the reference point lies, and the nodes' within the error of their
longest chain of additions."""
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


@pytest.mark.parametrize("precision", ("fp64", "fp32"))
@pytest.mark.parametrize("nw,ref", ((1, 8.25), (1023, 8.25), (16384, 0.0), (16385, -3e7), (50001, 1e3)))
def test_walker_sums_round_once(B, nw, ref, precision):
    n = (18, 15, 21)
    dom = W._domain(n, ("periodic",) * 3, 0.8, (1e-4, 0, 0), 0.1, seed=nw, u0=(0.05, -0.02, 0.01), precision=precision)
    g = B.build_domain(dict(domain=dom, walkers=dict(kind="uniform", n=nw, ref=(ref, ref, ref))))
    g.step(9)
    cell, off, img = g.walkers()
    c = np.stack([cell % n[0], (cell // n[0]) % n[1], cell // (n[0] * n[1])]).astype(np.int64)
    dv = ((c + img.astype(np.int64) * np.asarray(n)[:, None]).astype(float) - ref) + off
    for m in (g.moments(), g.moments(noalloc=True)):
        for a in range(3):
            for got, terms in ((m["sum"][a], dv[a]), (m["sumsq"][a], dv[a] * dv[a])):
                want = math.fsum(terms)
                # 2^-60 per term, and the final combination's three roundings
                assert abs(got - want) <= nw * 2.0 ** -60 + 4 * np.spacing(abs(want)), (a, got, want)


@pytest.mark.parametrize("n", ((3, 2, 2), (16, 16, 16), (17, 15, 16), (64, 64, 5), (5, 821, 5)))
def test_node_sums(B, n):
    dom = W._domain(n, ("periodic",) * 3, 0.8, (1e-4, 2e-4, 0), 0.1, seed=1, u0=(0.05, -0.02, 0.01))
    g = B.build_domain(dict(domain=dom))
    g.step(3)
    u, rho = g.velocity()
    m = g.moments()
    N = int(np.prod(n))
    gamma = 40 * 2.0 ** -53  # 4 nodes a thread, 6 + 16 folds, chunks, and the product's rounding
    assert abs(m["mass"] - math.fsum(rho.ravel())) <= gamma * np.abs(rho).sum()
    for a in range(3):
        t = (rho * u[a]).ravel()
        assert abs(m["momentum"][a] - math.fsum(t)) <= gamma * np.abs(t).sum()
        assert abs(m["fluid_u"][a] - math.fsum(u[a].ravel()) / N) <= 2 * gamma * np.abs(u[a]).sum() / N
    assert m["solid_volume"] == 0.0 and not m["particle_v"].any()
