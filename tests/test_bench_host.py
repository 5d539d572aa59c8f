"""Host-side checks of bench.py (no GPU): the one-GPU contract and the
counter-traffic bookkeeping."""
import os
import subprocess
import sys

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode == 2
    assert "one GPU" in res.stderr


def test_traffic_is_null_once_the_kernel_source_changes(monkeypatch):
    for kernel, (src, fetch, write) in bench.TRAFFIC_KIB.items():
        assert src in bench.TRAFFIC_SOURCES
        assert fetch > 0 and write >= 0
    monkeypatch.setitem(bench.TRAFFIC_SOURCES, "linear_decode.hip", "0" * 64)
    assert bench.traffic_bytes("gemv_lut_kernel<1,2,2>") is None
    assert bench.traffic_bytes("no_such_kernel") is None


def test_traffic_scale_from_copy_is_sane():
    # the counters were scaled by a plain copy: both factors near small integers
    assert 0.9 < bench.TRAFFIC_WRITE_SCALE < 1.1
    assert 0.9 < bench.TRAFFIC_FETCH_SCALE < 2.1


def test_the_line_keeps_the_headline_and_stays_short():
    row = {"levels": 3, "had": 1, "osr": 1.25, "bits_per_weight": 2.5, "out_rel_err": 1.2171897665549791,
           "weight_snr_db": -1.7200476517793215}
    line = {"metric": "m", "value": 5123.456789012345, "ms_per_step": 8.123456789012345,
            "config": {"a": 1.23456789, "b": [0.1234567891]},
            "phases": {"precision_sweep": {"rows": [dict(row) for _ in range(78)], "sweep_s": 0.1234567891}}}
    out = bench._short_line(line)
    assert out["value"] == line["value"] and out["ms_per_step"] == line["ms_per_step"]
    assert out["config"] == {"a": 1.23457, "b": [0.123457]}
    assert out["phases"]["precision_sweep"] == {"rows": 78, "sweep_s": 0.123457}
    assert len(line["phases"]["precision_sweep"]["rows"]) == 78       # the line itself is left as it is
