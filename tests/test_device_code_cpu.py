"""Checks of the device code in the built library that need no GPU."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2507_11512_amd", "libhpgmx.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def kernel_code(tmp_path, name):
    """The instructions of the kernel whose mangled name holds `name`."""
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    for f in glob.glob(str(tmp_path / "*gfx950")):
        syms = subprocess.run([OBJDUMP, "--syms", f], check=True, capture_output=True, text=True).stdout
        for sym in re.findall(r" F \.text\s.*\s(\S*" + name + r"\S*)$", syms, re.M):
            out = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + sym, f], check=True,
                                 capture_output=True, text=True).stdout
            return [line.split("//")[0].strip() for line in out.splitlines()]
    raise AssertionError(f"no kernel {name} in the library")


def test_scalars_are_released_to_the_host(tmp_path):
    """The host reads a step's scalars behind an event without a system fence, so the finish kernel itself has to
    write back to system scope and wait for it after its last store to them."""
    if not os.path.exists(LIB):
        pytest.fail("libhpgmx.so is not built; run __graft_entry__.build()")
    code = kernel_code(tmp_path, "k_finishE")
    stores = [i for i, c in enumerate(code) if c.startswith("global_store") and c.endswith("sc0 sc1")]
    runs = [i for i, j in zip(stores, stores[1:] + [len(code)]) if j - i > 20]  # last store of each group
    assert len(runs) == 3  # the Givens step, the residual's and the right-hand side's norm
    for i in runs:
        after = code[i + 1:i + 8]
        release = [j for j, c in enumerate(after) if c.startswith("buffer_wbl2 sc0 sc1")]
        assert release, after
        assert any(c.startswith("s_waitcnt") and "vmcnt(0)" in c for c in after[release[0] + 1:]), after
