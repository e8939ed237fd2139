"""What the built kernels wait for, from the assembly of their code objects: a payload that comes out of host memory
takes longer than everything else a launch asks for, and only what needs it may wait for it."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2411_03357_amd as pgcm
from test_kernel_scratch import _code_objects, _kernels

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_decrypting_rows_the_tables_are_not_waited_for_with_the_payload(tmp_path):
    """burst_kernel, decrypting in rows without sweeps (kinds 1 and 5): the row is the last thing asked for ahead of
    the first barrier, and behind it the tables are waited for with that one load still on its way"""
    with open(pgcm.library_path(), "rb") as f:
        image = f.read()
    seen = 0
    for n, elf in enumerate(_code_objects(image)):
        names = [k[".name"] for k in _kernels(elf)]
        names = [k for k in names if re.search(r"burst_kernelILb1ELb.ELNS_9BurstKindE[15]E", k)]
        if not names:
            continue
        path = tmp_path / ("object_%d" % n)
        path.write_bytes(elf)
        out = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--disassemble-symbols=" + ",".join(names), str(path)],
                             stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
        assert out.returncode == 0, out.stderr[-500:]
        for kernel in re.split(r"^[0-9a-f]+ <", out.stdout, flags=re.M)[1:]:
            name, code = kernel.split(">:", 1)
            code = [line.split("//")[0].strip() for line in code.splitlines()]
            barrier = code.index("s_barrier")
            loads = [c for c in code[:barrier] if c.startswith("global_load")]
            assert loads[-1].startswith("global_load_dwordx4"), (name, loads[-1])
            waits = [c for c in code[barrier:] if c.startswith("s_waitcnt") and "vmcnt" in c]
            assert int(re.search(r"vmcnt\((\d+)\)", waits[0]).group(1)) >= 1, (name, waits[0])
            seen += 1
    assert seen == 12, seen      # two lengths of IV, two kinds, three forms of arguments
