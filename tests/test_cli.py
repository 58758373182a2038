"""Command-line contract of the two benchmark scripts, as far as it can be checked without a GPU."""
import os
import subprocess
import sys

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(*argv):
    return subprocess.run([sys.executable, *argv], cwd=ROOT, capture_output=True, text=True, timeout=120)


@pytest.mark.parametrize("script", ["bench.py", "bench_table1.py"])
def test_help_renders(script):
    r = run(script, "--help")
    assert r.returncode == 0, r.stderr
    assert "usage" in r.stdout


def test_more_than_one_gpu_is_refused_with_a_message():
    r = run("bench.py", "--gpus", "2")
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


@pytest.mark.parametrize("l2s", [1, 2, 4, 8])
def test_traffic_bounds_hold_however_many_l2s_pull_the_code(l2s):
    """Data requests count as half their bytes, instruction fetches in full; how many L2s pull a block depends on the deal."""
    code, data, write = 1.5e6, 12e6, 12e6
    least, most = bench.traffic_bounds(l2s * code + data / 2, write, {"FETCH_SIZE": 2.0, "WRITE_SIZE": 1.0}, code)
    assert least <= l2s * code + data + write <= most
    assert least == l2s * code + data + write or l2s < 8
