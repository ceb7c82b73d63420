"""Read-outs large enough for several copy workers, on each kind of stream a
domain can have and beside other work on the device."""
import ctypes as C

import numpy as np
import pytest

from paper_2308_05007_amd import workloads as W

pytestmark = pytest.mark.gpu

PER_THREAD = 2  # the handle hipStreamPerThread: another stream in every thread


@pytest.fixture(scope="module")
def B():
    from paper_2308_05007_amd import binding
    binding.lib()
    return binding


def _cfg(n=(128, 128, 128), nw=1_000_000):
    dom = W._domain(n, ("periodic",) * 3, 0.8, (1e-5, 2e-5, 0), 0.05, seed=3, u0=(0.05, 0.02, -0.01), precision="fp32")
    return dict(domain=dom, walkers=dict(kind="uniform", n=nw, ref=tuple(v / 2 for v in n)))


def test_per_thread_stream(B, monkeypatch):
    cfg = _cfg()
    a = B.build_domain(cfg)
    make = B.make_desc

    def make_per_thread(*args):
        d = make(*args)
        d.stream = C.c_void_p(PER_THREAD)
        return d

    monkeypatch.setattr(B, "make_desc", make_per_thread)
    b = B.build_domain(cfg, use_torch=False)
    for read in (B.Domain.velocity, B.Domain.walkers, lambda d: (d.distributions(),)):
        a.step(300)
        b.step(300)  # still in the queue when the read-out is called
        for x, y in zip(read(a), read(b)):
            assert np.array_equal(x, y)
