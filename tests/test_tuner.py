"""The autotuners' decision, on planted times (CPU only; the timing itself needs
a GPU, see test_gpu_parity.py)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_02257_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_a_choice_is_entered_only_where_it_beats_no_choice(tmp_path):
    exe = tmp_path / "driver"
    srcs = [os.path.join(CSRC, "host", s) for s in ("dag.cpp", "kplan.cpp")] + [
        os.path.join(ROOT, "tests", "tuner", "driver.cpp")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                        *srcs, "-o", str(exe)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "tuner driver: ok" in r.stdout, r.stdout
