"""The fixed-order loops' lists on the host: tests/fixed_lists.cpp against the planner's
source, and opf_plan_verify over the plans that have them."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_1403_7209_amd as pk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1403_7209_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_lists_and_their_verification(tmp_path):
    exe = tmp_path / "fixed_lists"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                        "-I", CSRC, os.path.join(ROOT, "tests", "fixed_lists.cpp"),
                        os.path.join(CSRC, "planner.cpp"), "-o", str(exe), "-pthread"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    assert r.stdout.strip() == "ok"


@pytest.mark.parametrize("K", [0, 64, 512, 1024])
@pytest.mark.parametrize("N", [512, 3000, 98304, 98305])
def test_plan_verify_with_lists(N, K):
    i = np.arange(N - 1, dtype=np.int32)
    e2n = np.concatenate([np.stack([i, i + 1], 1), np.stack([i[3:], i[:-3]], 1)])
    ctx = pk.Context(None)
    nodes, edges = ctx.decl_set(N, "nodes"), ctx.decl_set(len(e2n), "edges")
    m = ctx.decl_map(edges, nodes, 2, e2n, 0, "e2n")
    ctx.plan(m, cluster_size=K)
    assert ctx.plan_verify(m)["ok"]
