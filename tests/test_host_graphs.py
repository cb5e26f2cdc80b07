"""Capture, replay, limit and end of a context's graphs, on the CPU stand-in of
the HIP runtime (tests/host_mock/graphs.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT = os.path.join(ROOT, "_build", "mock")
WRAPPED = ("hipGraphLaunch", "hipGraphExecDestroy", "hipStreamSynchronize", "hipDeviceSynchronize")


def _sh(*cmd):
    r = subprocess.run(cmd, cwd=ROOT, capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-3000:]
    return r.stdout


def test_graphs():
    if not shutil.which("/opt/rocm/bin/hipcc"):
        pytest.skip("no ROCm compiler")
    _sh("bash", "tests/host_mock/build.sh")
    _sh("bash", "tests/host_mock/link.sh", "graphs", *[f"-Wl,--wrap={f}" for f in WRAPPED])
    assert "graphs: 0 failed" in _sh(os.path.join(OUT, "graphs"))
