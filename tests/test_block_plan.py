"""Elimination plans of the block-sparse Cholesky (csrc/blockplan.h), executed
on the host over graphs of every shape the analysis can meet: paths, bands,
loops, dense, disconnected and single-pose systems, in their own and in a
shuffled base order, dissected and not."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2408_01654_amd", "csrc")


def test_plans_solve_their_systems(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "block_plan_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(HERE, "block_plan_check.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    # a long path or band is eliminated in far fewer steps than it has blocks
    rows = [line.split() for line in r.stdout.splitlines()]
    path = {row[row.index("split") + 1]: int(row[row.index("levels") + 1]) for row in rows
            if row[0] == "path" and row[2] == "120"}
    assert path["1"] * 2 < path["0"]
