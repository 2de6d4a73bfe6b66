"""The benchmark's default line holds its sub-records by their figures, so that it stays short (CPU only)."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def figures(*records):
    """in a process of its own: bench.py sets environment variables when it is imported"""
    r = subprocess.run([sys.executable, "-c", "import json, sys, bench\n"
                        "print(json.dumps([bench.figures(x) for x in json.load(sys.stdin)]))"],
                       input=json.dumps(records), capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


def test_figures_of_every_kind_of_sub_record():
    bulk = {"config": {"workload": "x" * 500}, "library_statistics": list(range(200)), "unit": "GB/s", "steps": 20}
    step = dict(bulk, value=54.5, ms_per_step=114.389, roofline={"frac": 0.98, "traffic": "y" * 300},
                step_time={"overhead_vs_noswap_pct": 95.2, "overhead_vs_floor_out_then_in_pct": 4.7},
                cpu_baseline={"value": 32.9, "sample": "z" * 300})
    torch_swap = dict(bulk, ms_per_step={"no_hook_no_swap": 32.2, "swapping": 43.3}, overhead_vs_no_swap_pct=34.4)
    reuse = dict(bulk, step_ms=124.4, device_side_release_ops={"mean": 8.7}, host_polled_release_ops={"mean": 161.2})
    hook = dict(bulk, shapes={"gpu_bound": {"modes": {"hook, Detailed mode": {"overhead_pct": 0.0}}}})
    got = figures(step, torch_swap, reuse, hook, {"failed": "SsError: " + "w" * 1000})
    assert got[0] == {"ms": 114.389, "value": 54.5, "overhead_pct": 95.2, "over_floor_pct": 4.7, "roofline_frac": 0.98,
                      "cpu_value": 32.9}
    assert got[1] == {"ms": 43.3, "overhead_pct": 34.4}
    assert got[2] == {"ms": 124.4, "device_release_ops": 8.7, "host_release_ops": 161.2}
    assert got[3] == {"gpu_bound_detailed_pct": 0.0}
    assert got[4]["failed"].startswith("SsError") and max(len(json.dumps(x)) for x in got) < 150
