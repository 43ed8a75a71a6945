"""Host memory running out inside opf_plan: tests/oom_plan.cpp, linked against
libopflux.so, makes one allocation after another fail and expects a status, never an
exception or an abort."""
import os
import shutil
import subprocess

import pytest

import paper_1403_7209_amd as pk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_out_of_host_memory_is_a_status(tmp_path):
    lib = pk.LIB_PATH
    assert os.path.exists(lib), "libopflux.so is not built"
    exe = tmp_path / "oom_plan"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "oom_plan.cpp"), "-o", str(exe), lib,
                        f"-Wl,-rpath,{os.path.dirname(lib)}", "-pthread"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert r.stdout.strip() == "ok"
