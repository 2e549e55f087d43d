"""CPU-only: how the built kernels form the addresses of buffer instructions, from the library's own code objects."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_13989_amd import binding
from test_kernel_registers import _code_objects

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def test_buffer_instructions_have_no_scalar_offset(tmp_path):
    """Rows are bounded by the range check of a buffer resource (narrow rows read zero beyond their width), and the scalar offset is
    not part of what it compares: every offset is in the vector register or in the instruction."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not found")
    binding.lib()
    path, count = str(tmp_path / "a.co"), 0
    for obj in _code_objects():
        with open(path, "wb") as f:
            f.write(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout
        for line in re.findall(r"\bbuffer_(?:load|store|atomic)_\w+ [^/\n]*", text):
            # data, vector offset, resource, scalar offset and flags
            operands = [o.strip() for o in line.split(" ", 1)[1].split(",")]
            assert operands[3].split()[0] == "0", line
            count += 1
    assert count > 5000
