"""What the built kernels may not contain, read from the disassembly of the
library's own gfx950 code: binary64 arithmetic (every accumulation is binary32
or integer; binary64 is the CPU oracle's) and packed binary32 instructions."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_22228_amd import pcoll as pc

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump",
                            shutil.which("llvm-objdump") or "")
                if p and os.path.exists(p)), None)


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_kernels_use_no_binary64(tmp_path):
    pc.load()
    lib = shutil.copy(pc.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, cwd=tmp_path,
                   capture_output=True)
    objs = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert objs
    found = {}
    for f in objs:
        p = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", f],
                             cwd=tmp_path, stdout=subprocess.PIPE, text=True)
        ops = 0
        for line in p.stdout:
            m = re.match(r"\s+([a-z]\w+)", line)
            if not m:
                continue
            ops += 1
            op = m.group(1)
            if "f64" in op or re.match(r"v_pk_(add|mul|fma)_f32", op):
                found[op] = found.get(op, 0) + 1
        assert p.wait() == 0
        assert ops > 100, f
    assert not found, found
