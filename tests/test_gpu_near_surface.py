"""Near-surface walkers against the FP64 oracle, bit for bit, where a block's
queue and a row's control points change form: particles of fewer, exactly and
more than 16 control points (a row of lanes holds 16 at a time), two particles
whose mask words overlap, few and many walkers whose step ends inside."""
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


@pytest.mark.parametrize("walls", (False, True))
@pytest.mark.parametrize("n_walkers", (40, 2500))
@pytest.mark.parametrize("nc", (1, 15, 16, 17, 33, 64))
def test_near_surface_rows(orc, B, nc, n_walkers, walls):
    rng = np.random.default_rng(100 * nc + n_walkers)
    n = (14, 13, 15)
    parts = []
    for i, x in enumerate((4.5, 9.5)):
        b, k = W.metaball_shape(rng, nc if i == 0 else max(1, nc // 2), 1.0, (0.5, 1.0))
        parts.append(dict(b=b, k=k * (4.0 / k.sum()), centre=np.array([x, 6.5, 7.0]), motion="sinusoid",
                          amp=np.array([1.5, 0.4, 0.0]), period=25.0, phase=0.2 * i))
    dom = W._domain(n, ("periodic", "wall" if walls else "periodic", "periodic"), 0.8, (1e-5, 0, 0), 0.2, seed=nc)
    cfg = dict(domain=dom, particles=parts, walkers=dict(kind="uniform", n=n_walkers, ref=(7.0, 6.5, 7.5)))
    o, g = _pair(orc, B, cfg)
    for _ in range(3):
        o.step(4)
        g.step(4)
        compare(o, g)
    c = g.moments()["counters"]
    if n_walkers > 1000:
        assert c["type4"] > 100 and c["type2"] > 20, c
