"""Where the kernels of the built library start: each on a page of its own (the build says what it is worth)."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2604_23108_amd as M

LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objdump"), reason="needs the compiler's llvm-objdump and llvm-readelf")
def test_kernels_start_on_pages(tmp_path):
    lib = shutil.copy(M.lib_path(), tmp_path / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    starts = {}
    for code in sorted(tmp_path.glob("lib.so.*gfx950*")):
        out = subprocess.run([f"{LLVM}/llvm-readelf", "-s", "-W", str(code)], check=True, capture_output=True, text=True).stdout
        # functions of the code object: value, size, ..., name
        starts.update({m.group(2): int(m.group(1), 16) for m in re.finditer(r":\s+([0-9a-f]{16})\s+\d+\s+FUNC\s.*\s(\S+)\n", out)})
    assert len(starts) > 100
    assert not {n: hex(a) for n, a in starts.items() if a % 4096}
