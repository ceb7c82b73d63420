"""Bytes the benchmark credits where fluid updates are taken two per pass."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


@pytest.mark.parametrize("nw", (0, 10_000_000))
def test_paired_updates_share_a_read_and_a_write(nw):
    """88 bytes per node and paired update (19 reads, 19 writes for two, three
    velocity components each), 164 per single one, with walkers and without."""
    import bench
    from paper_2308_05007_amd import workloads as W
    cfg = W.config_oscillator(precision="fp32", n_walkers=10_000_000)
    cfg["walkers"]["n"] = nw
    N = 256 ** 3
    assert bench.credited_bytes(cfg, "fp32", 100, 100, 100) == 100 * (88 * N + 32 * nw)
    assert bench.credited_bytes(cfg, "fp32", 101, 101, 100) == (100 * 88 + 164) * N + 101 * 32 * nw
    assert bench.credited_bytes(cfg, "fp32", 1, 1, 0) == 164 * N + 32 * nw


@pytest.mark.parametrize("nw", (0, 10_000_000))
@pytest.mark.parametrize("paired", (0, 64))
def test_the_record_decides_not_the_launch_counts(monkeypatch, nw, paired):
    import bench
    from paper_2308_05007_amd import workloads as W
    cfg = W.config_oscillator(precision="fp32", n_walkers=10_000_000)
    cfg["walkers"]["n"] = nw
    launches = (32 if not nw else 96) if paired else 65
    monkeypatch.setattr(bench, "run_plain", lambda *a, **k: (
        1.0, (20.0, launches, 64, 64 if nw else 0, paired), dict(n_walkers=nw)))
    r = bench.measure(cfg, "k", 64, 0, 32)
    want = 64 * ((88 if paired else 164) * 256 ** 3 + 32 * nw)
    assert r["achieved"] == pytest.approx(want / 0.02 / 1e9, rel=1e-12)
    assert ("k_pair" in r["kernel"]) == bool(paired)
