"""LDS of the allocation-free application's kernel: the forces take the place of the
staged D rows, each lane's over rows that other lanes read, so a barrier has to lie
between a block's last read of D and its first force.  Looked for in the code that was
built (in source order the compiler may move either past the other)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
@pytest.mark.parametrize("mode", [0, 1])  # A and K: the operators that read D
def test_barrier_between_staged_rows_and_forces(nlth_mod, tmp_path, mode):
    so = shutil.copy(nlth_mod.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", so], cwd=tmp_path, check=True, capture_output=True)
    listing = ""
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" in f:
            syms = subprocess.run([OBJDUMP, "-t", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
            name = re.search(r"\.text\s.*\s(_ZN4nlth12k_op_input64ILi%dE\S+)$" % mode, syms, re.M)
            if name:
                listing = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + name.group(1), f], cwd=tmp_path,
                                         check=True, capture_output=True, text=True).stdout
    ops = re.findall(r"^\s+(s_barrier|ds_read\w*|ds_write\w*)\b", listing, re.M)
    # staging (writes), barrier, D rows and nodal values (reads), barrier, forces
    # (writes), barrier, row sums (reads)
    parts, cur = [], set()
    for op in ops:
        if op == "s_barrier":
            parts.append(cur)
            cur = set()
        else:
            cur.add("read" if op.startswith("ds_read") else "write")
    parts.append(cur)
    print(mode, parts)
    assert parts == [{"write"}, {"read"}, {"write"}, {"read"}]
