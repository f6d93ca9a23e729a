"""Host-side behaviour of bench.py that needs no GPU."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_cpu_baseline_sample_is_bounded():
    """The CPU leg takes every tree of a small workload and a sample of whole trees of a large one."""
    sys.path.insert(0, ROOT)
    import bench
    from paper_1809_00832_amd import synth
    small = bench.cpu_baseline(synth.workload("tiny"))
    assert small["kind"] == "oracle" and small["unit"] == "trees/s" and small["value"] > 0 and "all 4 trees" in small["sample"]
    big = bench.cpu_baseline(synth.workload("sentence"), max_nodes=300)
    assert "of the 25 trees" in big["sample"] and big["cores"] >= 1


def test_the_line_on_stdout_is_short_and_complete():
    """What other schedulers, workloads and training steps were measured at does not go into the headline line."""
    import json
    sys.path.insert(0, ROOT)
    import bench
    keys = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
            "config", "roofline", "stage_ms", "cpu_baseline")
    out = {k: 0.123456789012345 for k in keys}
    out["roofline"] = {"k%d" % i: 0.123456789012345 for i in range(12)}
    out["cpu_baseline"] = bench.cpu_baseline(__import__("paper_1809_00832_amd.synth", fromlist=["x"]).workload("tiny"))
    for k in bench.HEADLINE_LEAVES_OUT:
        out[k] = ["x" * 100] * 100
    line = json.dumps(bench.headline(out))
    assert len(line) < 3000
    assert set(keys) == set(json.loads(line))


@pytest.mark.parametrize("workload, scheduler, precision, terms", [
    ("throughput", "dataflow", "f32", 3), ("throughput", "level_device", "f32", 0), ("treernn", "dataflow", "f32", 3),
    ("treernn", "ready", "f32", 0), ("rntn", "dataflow", "f32", 3), ("rntn", "level_host", "f32", 3), ("treernn", "dataflow", "bf16", 1)])
def test_rate_of_the_unit_that_does_the_products(workload, scheduler, precision, terms):
    """The rate that a kernel's products are set against is that of the unit they run on: set against the fp32
    instructions' rate, RNTN came out above it."""
    import bench
    want = bench.PEAK_TFLOPS["bf16"] / terms if terms else bench.PEAK_TFLOPS["f32"]
    assert bench.matrix_peak(workload, scheduler, precision) == want
