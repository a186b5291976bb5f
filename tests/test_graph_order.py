"""Dependencies of the graph that issue mode 2 is added to (CPU only).

The walk over a plan's steps and the bookkeeping of the graph's nodes
(runtime/walk.hpp, runtime/graph_order.hpp) are plain C++; they are compiled
with g++ into tests/graph_order/driver.cpp, which records nodes and edges in
place of a HIP graph.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_02257_amd", "csrc")
HOST = ["host/dag.cpp", "host/sched.cpp", "host/plan.cpp", "host/kplan.cpp", "capi.cpp"]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_graph_nodes_are_one_sequence_without_copies_and_ordered_with_them(tmp_path):
    exe = tmp_path / "driver"
    srcs = [os.path.join(CSRC, s) for s in HOST] + [
        os.path.join(ROOT, "tests", "sanitize", "device_stub.cpp"),
        os.path.join(ROOT, "tests", "graph_order", "driver.cpp")]
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Wno-unused-parameter", "-I", CSRC,
           "-I", os.path.join(ROOT, "include"), *srcs, "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "warning" not in r.stderr, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "graph order driver: ok" in r.stdout, r.stdout[-3000:] + r.stderr[-2000:]
