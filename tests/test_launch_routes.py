"""The host's choice of kernels, on the CPU (launch_trace.cpp).  Over a grid of shapes, chunk sizes, alignments and length promises, every operand of a backward contraction
is an input or an array that an earlier launch of the same call wrote, and none that reads an input writes a gradient in its place.  The residual-VQ encode takes the kernel
that is measurably the faster one."""
import os
import shutil
import subprocess

import pytest

from paper_2603_16435_amd import binding

SOURCE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_trace.cpp")
pytestmark = pytest.mark.skipif(not os.path.exists(binding.LIB_PATH) or not shutil.which("g++"), reason="library not built, or no g++")


@pytest.fixture(scope="module")
def trace(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("trace") / "launch_trace")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-o", exe, SOURCE, "-ldl"], check=True)
    return lambda *args: subprocess.run([exe, binding.LIB_PATH, *map(str, args)], capture_output=True, text=True, timeout=100)


def test_every_operand_of_a_contraction_is_made_by_the_call(trace):
    run = trace()
    assert run.returncode == 0, run.stdout + run.stderr
    for kind in ("bf16 pair", "dW", "dX", "dX K-major", "small grads", "small pair"):          # the grid reaches all of them
        assert f"\n{kind}: " in run.stdout, run.stdout


# groups, vectors of each, stages, entries: us of the kernel for few vectors, of the one for many, where one takes at least a fifth longer whether or not the second
# has to look at a stage again
ENCODE = [
    (512, 256, 2, 64, 172, 31), (264, 512, 2, 64, 179, 53), (64, 1024, 2, 64, 90, 31), (100, 512, 1, 512, 85, 33), (64, 700, 1, 512, 75, 33),
    (128, 200, 1, 512, 50, 23), (128, 256, 8, 64, 123, 54), (64, 400, 8, 64, 119, 71), (64, 400, 8, 128, 126, 86), (2048, 128, 2, 64, 334, 180),
    (512, 160, 24, 768, 2366, 776), (4096, 128, 10, 256, 3061, 1120),
    (8, 1024, 8, 64, 36, 77), (12, 17, 10, 256, 47, 75), (1, 17, 40, 256, 162, 280), (37, 17, 40, 256, 165, 365), (12, 512, 32, 64, 111, 269), (1024, 32, 8, 512, 278, 401),
]


def test_encode_takes_the_faster_kernel(trace):
    run = trace(*(x for c in ENCODE for x in c[:4]))
    assert run.stdout.split() == ["few" if c[4] < c[5] else "many" for c in ENCODE], list(zip(ENCODE, run.stdout.split()))
