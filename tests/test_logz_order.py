"""The last workgroup of the log-Z head's hidden layer reads sums that other workgroups wrote, on other dies: in the library as it is built, the count that announces
a sum is a release and an acquire at the scope of the device (what an L2 holds is written back ahead of it, and dropped behind it)."""
import os
import re
import subprocess

import pytest

from paper_2603_16435_amd import binding
from test_hot_loop_loads import TOOLS


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH) or not all(map(os.path.exists, TOOLS)), reason="library or LLVM tools not there")
def test_the_count_of_the_hidden_layer_is_a_release_and_an_acquire(tmp_path):
    copy, unbundle, dump = TOOLS
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev.o")
    subprocess.run([copy, f"--dump-section=.hip_fatbin={fat}", binding.LIB_PATH, os.devnull], check=True)
    subprocess.run([unbundle, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={dev}"], check=True)
    text = subprocess.run([dump, "-d", "--no-show-raw-insn", "--no-leading-addr", dev], check=True, capture_output=True, text=True).stdout
    kernels = [f for f in re.split(r"\n(?=[0-9a-f]* ?<)", text) if re.match(r"[0-9a-f]* ?<[^>]*logz_hidden_kernel", f)]
    assert len(kernels) == 2
    for f in kernels:
        ins = [line.split("//")[0].strip() for line in f.splitlines()]
        at = [i for i, s in enumerate(ins) if s.startswith("global_atomic_add")]
        assert len(at) == 1
        before, behind = ins[at[0] - 12:at[0]], ins[at[0]:at[0] + 12]
        assert any(re.match(r"buffer_wbl2.*sc1", s) for s in before) and any(re.match(r"buffer_inv.*sc1", s) for s in behind), before + behind
