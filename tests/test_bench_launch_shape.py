"""The benchmark's stored HBM counters belong to one launch shape: 48 steps of
four-wave regions at 16 points per thread.  Other points or waves have other
rims and traffic, so they get none."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_counters_only_for_the_measured_shape():
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    assert "paper_1911_05769_amd/csrc/at_wave.h" in b.TRAFFIC["sources"]    # the exchange
    r = {"s": b.TRAFFIC["fuse"], "arith": 0, "ppt": 16, "waves": 4}
    saved = dict(b.TRAFFIC)
    try:
        b.TRAFFIC.update(md5=b.sources_md5(b.TRAFFIC["sources"]), bytes_per_launch=5.0)
        assert b.measured_traffic(r) == 5
        assert b.measured_traffic(dict(r, ppt=32, waves=1)) is None
        assert b.measured_traffic(dict(r, waves=1)) is None
    finally:
        b.TRAFFIC.clear()
        b.TRAFFIC.update(saved)
