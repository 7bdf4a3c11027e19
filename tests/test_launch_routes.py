"""The host's choice of kernels, on the CPU: over a grid of shapes, chunk sizes, alignments and length promises, every operand of a backward contraction is an
input or an array that an earlier launch of the same call wrote, and none that reads an input writes a gradient in its place (launch_trace.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_2603_16435_amd import binding

SOURCE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_trace.cpp")


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH) or not shutil.which("g++"), reason="library not built, or no g++")
def test_every_operand_of_a_contraction_is_made_by_the_call(tmp_path):
    exe = str(tmp_path / "launch_trace")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-o", exe, SOURCE, "-ldl"], check=True)
    run = subprocess.run([exe, binding.LIB_PATH], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout + run.stderr
    for kind in ("bf16 pair", "dW", "dX", "dX K-major", "small grads", "small pair"):          # the grid reaches all of them
        assert f"\n{kind}: " in run.stdout, run.stdout
