"""Read-outs of each size class (straight, through a host buffer, in chunks by
several workers with a last one that is not whole) against the
FP64 oracle, bit for bit, and read-outs of a part of what a call can return."""
import ctypes as C

import numpy as np
import pytest
from test_gpu_parity import _pair, compare

from paper_2308_05007_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2308_05007_amd import binding
    binding.lib()
    return binding


def _cfg(n, nw, precision="fp64"):
    rng = np.random.default_rng(nw)
    b, k = W.metaball_shape(rng, 5, 2.0, (0.5, 1.0))
    parts = [dict(b=b, k=k, centre=np.array([v / 2 for v in n]), motion="sinusoid", amp=np.array([2.0, 0, 0]),
                  period=50.0, phase=0.1)]
    dom = W._domain(n, ("periodic",) * 3, 0.8, (1e-5, 0, 0), 0.05, seed=3, precision=precision)
    return dict(domain=dom, particles=parts, walkers=dict(kind="uniform", n=nw, ref=tuple(v / 2 for v in n)))


@pytest.mark.parametrize("n,nw", (((20, 17, 23), 900), ((40, 31, 37), 60_001), ((70, 61, 83), 300_007)))
def test_readouts_of_every_size(orc, B, n, nw):
    o, g = _pair(orc, B, _cfg(n, nw))
    o.step(3)
    g.step(3)
    compare(o, g)


@pytest.mark.parametrize("precision", ("fp64", "fp32"))
def test_partial_readouts(B, precision):
    n, nw = (70, 61, 83), 300_007
    g = B.build_domain(_cfg(n, nw, precision))
    g.step(2)
    u, rho = g.velocity()
    cell, off, img = g.walkers()
    vp = lambda a: a.ctypes.data_as(C.c_void_p)
    u2, r2 = np.empty(u.size), np.empty(rho.size)
    assert g.L.rwmi_read_velocity(g.h, vp(u2), None) == 0
    assert g.L.rwmi_read_velocity(g.h, None, vp(r2)) == 0
    assert g.L.rwmi_read_velocity(g.h, None, None) == 0
    assert np.array_equal(u2, u.ravel()) and np.array_equal(r2, rho.ravel())
    c2, o2, i2 = np.empty_like(cell), np.empty_like(off), np.empty_like(img)
    assert g.L.rwmi_read_walkers(g.h, None, vp(o2), None) == 0
    assert g.L.rwmi_read_walkers(g.h, vp(c2), None, vp(i2)) == 0
    assert g.L.rwmi_read_walkers(g.h, None, None, None) == 0
    assert np.array_equal(c2, cell) and np.array_equal(o2, off) and np.array_equal(i2, img)
