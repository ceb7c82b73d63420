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


def test_readouts_do_not_wait_for_other_domains(B):
    """A read-out waits for its own domain's stream: another domain's queue
    (some 300 ms) is still running when a read-out of a few ms returns, the
    first of the process's as well as later ones."""
    other = B.build_domain(_cfg((256, 256, 256), 1_000))
    other.step(4)
    other.sync()
    a = B.build_domain(_cfg())
    a.step(2)
    for read in (B.Domain.velocity, B.Domain.walkers, B.Domain.distributions):
        a.sync()
        other.step(800)
        read(a)
        assert not other._torch_stream.query(), "the read-out waited for the whole device"
        other.sync()


def test_concurrent_readouts(B):
    """More read-outs at a time than there are pinned buffers."""
    import threading
    cfg = _cfg()
    doms = [B.build_domain(cfg) for _ in range(6)]
    for d in doms:
        d.step(3)
    want = doms[0].velocity()
    got = [None] * len(doms)

    def work(i):
        for _ in range(3):
            got[i] = doms[i].velocity()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(doms))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for u, rho in got:
        assert np.array_equal(u, want[0]) and np.array_equal(rho, want[1])
    for d in doms:
        d.close()
