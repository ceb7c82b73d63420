"""Which domains take their fluid steps in pairs, and that those which do have
the values of single steps, bit for bit: with and without particles and
walkers, the most particles, narrow tiles, planes of whole and of broken layout
tiles."""
import numpy as np
import pytest
from test_gpu_pairs import _same

from paper_2308_05007_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2308_05007_amd import binding
    binding.lib()
    return binding


def _cfg(n, np_, nw, force, points=(3, 7), radius=(2.0, 4.0), **kw):
    rng = np.random.default_rng(n[0])
    parts = []
    for i in range(np_):
        b, k = W.metaball_shape(rng, int(rng.integers(*points)), rng.uniform(*radius), (0.3, 1.2), rotate=True)
        parts.append(dict(b=b, k=k, centre=rng.uniform(size=3) * n, motion="sinusoid", amp=np.array([2.0, 1.0, 2.0]),
                          period=40.0, phase=float(rng.uniform())))
    dom = W._domain(n, kw.pop("bc", ("periodic",) * 3), 0.8, (2e-5, -1e-5, 1e-5) if force else (0, 0, 0), 0.01, seed=5,
                    u0=(0.02, -0.01, 0.015), precision=kw.pop("precision", "fp32"), **kw)
    c = dict(domain=dom, particles=parts)
    return dict(c, walkers=dict(kind="uniform", n=nw, ref=tuple(v / 2 for v in n))) if nw else c


@pytest.mark.parametrize("n,np_,nw,force", (((192, 192, 160), 0, 0, True), ((192, 192, 160), 0, 30_000, False),
                                            ((256, 256, 200), 64, 30_000, True), ((48, 48, 2600), 2, 10_000, False),
                                            ((250, 250, 125), 3, 10_000, True), ((1000, 121, 64), 5, 0, False),
                                            ((40, 370, 370), 0, 1000, True)))
def test_paired_updates_equal_single_ones(B, n, np_, nw, force):
    cfg = _cfg(n, np_, nw, force)
    a, b = B.build_domain(cfg), B.build_domain(cfg)
    taken = 0
    for steps in (5, 4, 1, 2):
        a.step(steps)
        taken += steps // 2 * 2
        assert a.paired() == taken
        for _ in range(steps):
            b.step(1)
        _same(a, b)
    assert b.paired() == 0


def test_graphs_and_timing_count_pairs(B):
    a = B.build_domain(_cfg((192, 192, 160), 0, 1000, False))
    a.set("use_graph", 1)
    a.step(261)  # two replays of 128 and 5 single launches' worth
    assert a.paired() == 260
    a.step(5)
    assert a.paired() == 264
    a.set("timing", 4)
    a.kernel_times()
    a.step(7)
    assert a.paired() == 270
    ms, launches, fluid, walkers = a.kernel_times()
    assert (launches, fluid, walkers) == (3 + 8 - 1, 7, 7)  # the first launch carries nothing


@pytest.mark.parametrize("why,cfg", (
    ("in place", dict(n=(170, 160, 160))),
    ("walls", dict(n=(192, 192, 160), bc=("periodic", "wall", "periodic"))),
    ("16-bit storage", dict(n=(256, 256, 200), precision="fp16")),
    ("particles that are the slower in pairs", dict(n=(192, 192, 160), np_=30, points=(50, 61), radius=(12.0, 14.0))),
    ("narrow tiles", dict(n=(16, 16, 21000))),
    ("narrow tiles whose rows begin anywhere", dict(n=(37, 64, 2300), nw=1000, force=True)),
))
def test_refused(B, why, cfg):
    g = B.build_domain(_cfg(**dict(dict(np_=0, nw=0, force=False), **cfg)))
    g.step(4)
    assert g.paired() == 0, why


def test_streamed_in_place_on_request(B):
    g = B.build_domain(_cfg((192, 192, 160), 0, 0, False))
    g.set("streaming", 2)
    g.step(4)
    assert g.paired() == 0
