"""The wait at the end of a slab of the bf16 hot kernel leaves one load in flight and relies on that being the L2 prefetch.  The source holds the
prefetch behind the slab's loads and ahead of the wait; here the library as it is built: a load into a register (the slab's go to LDS) is the
last vector memory operation before each such wait."""
import os
import re
import subprocess

import pytest

from paper_2603_16435_amd import binding

LLVM = "/opt/rocm/llvm/bin"
TOOLS = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH) or not all(map(os.path.exists, TOOLS)), reason="library or LLVM tools not there")
def test_the_prefetch_is_the_last_load_before_each_wait_that_leaves_one_in_flight(tmp_path):
    copy, unbundle, dump = TOOLS
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev.o")
    subprocess.run([copy, f"--dump-section=.hip_fatbin={fat}", binding.LIB_PATH, os.devnull], check=True)
    subprocess.run([unbundle, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={dev}"], check=True)
    text = subprocess.run([dump, "-d", "--no-show-raw-insn", "--no-leading-addr", dev], check=True, capture_output=True, text=True).stdout
    waits = 0
    last = ""                                            # last vector memory operation
    ins = [line.split("//")[0].strip() for line in text.splitlines()]
    for this, following in zip(ins, ins[1:]):
        if re.match(r"(global|buffer|flat|scratch)_", this):
            last = this
        elif this == "s_waitcnt vmcnt(1) lgkmcnt(0)" and following.startswith("s_barrier"):
            waits += 1
            assert last.startswith("global_load_dword "), last
    assert waits >= 2 * 8                                # two slabs per turn of the loop, eight kernels at the least


@pytest.mark.skipif(not os.path.exists(binding.LIB_PATH) or not all(map(os.path.exists, TOOLS)), reason="library or LLVM tools not there")
def test_the_narrow_f32_tiles_wait_for_their_loads_where_they_store_them(tmp_path):
    """The general kernel exchanges the middle elements of what it loads on the way to LDS.  Where the compiler does that ahead of the MFMAs, each wait for a load with a
    copy behind it is hundreds of instructions ahead of the store, and the loads are in flight for nothing."""
    copy, unbundle, dump = TOOLS
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev.o")
    subprocess.run([copy, f"--dump-section=.hip_fatbin={fat}", binding.LIB_PATH, os.devnull], check=True)
    subprocess.run([unbundle, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={dev}"], check=True)
    text = subprocess.run([dump, "-d", "--no-show-raw-insn", dev], check=True, capture_output=True, text=True).stdout
    met = held = 0
    for f in re.split(r"\n(?=[0-9a-f]+ <)", text):
        if not re.match(r"[0-9a-f]+ <\S*(gemm_nt_kernelIf\S*ELi16ELi\d+ELi1E|gemm_nt_small_pair_kernel)", f):
            continue
        both = re.match(r"[0-9a-f]+ <\S*EpiFwd\S*ELi256ELi16ELi4ELi1ELi1ELb1E", f)           # has a form that waits at once as well
        ins = [line.split("//")[0].strip() for line in f.splitlines()[1:]]
        for i, (this, following) in enumerate(zip(ins, ins[1:])):
            if this.startswith("s_waitcnt vmcnt") and re.match(r"v_mov_b32_e32 v\d+, v\d+", following):
                met += 1
                ok = any(s.startswith("ds_write_b128") for s in ins[i:i + 20])
                held += bool(both) and ok
                assert ok or both, (f.splitlines()[0], ins[i:i + 20])
    assert met >= 20 and held >= 2 * 4
