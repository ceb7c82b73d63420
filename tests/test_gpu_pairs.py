"""Fluid steps taken in pairs give the values of single steps, bit for bit: a
lattice large enough for pairs is advanced by one call of n steps (pairs, with
a single last step when n is odd) and by n calls of one (never paired).  Rows
that fill the tiles and rows that do not, planes of whole and of broken layout
tiles, body force, captured graphs, and mixtures of both kinds of call."""
import numpy as np
import pytest

from paper_2308_05007_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2308_05007_amd import binding
    binding.lib()
    return binding


def _cfg(n, force):
    rng = np.random.default_rng(n[0])
    shapes = [W.metaball_shape(rng, int(rng.integers(4, 13)), rng.uniform(3.0, 7.0), (0.3, 1.2), rotate=True)
              for _ in range(30)]
    centres = W.place_particles(rng, n, shapes, 3.0, (False,) * 3, tries=2000, allow_fewer=True)
    parts = [dict(b=b, k=k, centre=c, motion="sinusoid", amp=np.array([3.0, 1.0, 2.0]), period=60.0,
                  phase=float(rng.uniform())) for (b, k), c in zip(shapes, centres)]
    parts[0]["centre"] = np.array([0.3, 0.1, n[2] - 0.2])  # across three periodic faces
    dom = W._domain(n, ("periodic",) * 3, 0.8, (2e-5, -1e-5, 1e-5) if force else (0, 0, 0), 0.01, seed=5,
                    u0=(0.02, -0.01, 0.015), precision="fp32")
    return dict(domain=dom, particles=parts, walkers=dict(kind="uniform", n=200_000, ref=tuple(v / 2 for v in n)))


def _same(a, b):
    for x, y in zip((*a.velocity(), *a.walkers(), a.occupancy()), (*b.velocity(), *b.walkers(), b.occupancy())):
        assert np.array_equal(x, y)
    assert np.array_equal(a.distributions(), b.distributions())
    ma, mb = a.moments(), b.moments()
    assert all(np.array_equal(ma[k], mb[k]) for k in ("sum", "sumsq", "mass", "momentum", "fluid_u", "particle_v",
                                                      "solid_volume", "counters", "near_surface"))


@pytest.mark.parametrize("n,force", (((192, 192, 160), False), ((256, 136, 168), True), ((250, 250, 100), False),
                                     ((1000, 121, 64), True)))
def test_pairs_equal_single_steps(B, n, force):
    cfg = _cfg(n, force)
    a, b = B.build_domain(cfg), B.build_domain(cfg)
    for steps in (7, 2, 4):
        a.step(steps)
        for _ in range(steps):
            b.step(1)
        _same(a, b)


def test_pairs_in_graphs(B):
    cfg = _cfg((192, 192, 160), False)
    a, b = B.build_domain(cfg), B.build_domain(cfg)
    a.set("use_graph", 1)
    for steps in (5, 5, 6, 5, 1, 5):  # an odd number of lattice swaps per replay and an even one
        a.step(steps)
        for _ in range(steps):
            b.step(1)
    _same(a, b)
