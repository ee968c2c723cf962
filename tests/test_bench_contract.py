"""bench.py's command-line contract, as far as it can be checked without a GPU; the JSON line
itself is checked on the GPU."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr
    assert r.stdout.strip() == ""


def test_the_counted_traffic_belongs_to_the_present_kernels():
    sys.path.insert(0, ROOT)
    import bench
    assert bench.code_digest(bench.KERNEL_SOURCE) == bench.COUNTED_TRAFFIC["code_sha256"]


@pytest.mark.gpu
def test_json_line_has_the_agreed_fields():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--steps", "20", "--warmup", "5",
                        "--workload", "transformer_base"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [l for l in r.stdout.splitlines() if l.startswith("{")]
    assert len(lines) == 1
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better",
                "scaling", "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 20 and d["warmup"] == 5 and d["unit"] == "GB/s"
    assert d["config"]["workload"] == "transformer_base" and "model" not in d["config"]
    assert d["vs_baseline"] is None and d["data"] == "synthetic" and d["higher_is_better"] is True
    rf = d["roofline"]
    assert rf["bound"] == "hbm" and rf["peak"] == 8000.0 and rf["unit"] == "GB/s"
    assert abs(rf["frac"] - rf["achieved"] / rf["peak"]) < 1e-3 and "traffic" in rf
    cb = d["cpu_baseline"]
    assert cb["kind"] == "oracle" and cb["cores"] == 1 and cb["value"] > 0 and "sample" in cb
    assert d["parity_ok"] is True
    assert abs(d["value"] - d["algorithmic_bytes_per_step"] / (d["ms_per_step"] * 1e-3) / 1e9) < 1.0
