"""What the built kernels ask for at their start: one number of every cache line of their argument, all of it inside the struct that
the host fills in."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2007_06000_amd import binding as B
from test_matrix_operation_waits import OBJDUMP, functions

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(READELF)), reason="no disassembler")
def test_lines_asked_for_at_the_start_lie_inside_the_argument(tmp_path):
    lib = shutil.copy(B.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    seen = 0
    for part in sorted(tmp_path.glob("*gfx950")):
        notes = subprocess.run([READELF, "--notes", str(part)], check=True, capture_output=True, text=True).stdout
        size = {}       # of the struct that a kernel takes by value
        for kernel in notes.split("  - .agpr_count:")[1:]:
            given = re.findall(r"\.offset:\s+(\d+)\s+\.size:\s+(\d+)\s+\.value_kind:\s+by_value", kernel)
            name = re.search(r"^    \.name:\s+(\S+)$", kernel, re.M)[1]
            size[name] = max((int(o) + int(n) for o, n in given), default=0)
        listing = subprocess.run([OBJDUMP, "-d", str(part)], check=True, capture_output=True, text=True).stdout
        for name, ins in functions(listing):
            # the longest run of single loads, 64 bytes apart, from one address
            lines, run, base = [], [], None
            for op, args, _, _ in ins:
                m = re.match(r"\w+, (s\[\d+:\d+\]), (0x[0-9a-f]+|0)$", args) if op == "s_load_dword" else None
                at = int(m[2], 16) if m else None
                run = run + [at] if run and m and (m[1], at) == (base, run[-1] + 64) else [0] if at == 0 else []
                base = m[1] if m else None
                lines = max(lines, run, key=len)
            if size.get(name, 0) < 400:
                continue
            seen += 1
            assert lines and lines[-1] + 4 <= size[name] <= lines[-1] + 64, (name, lines, size[name])
    assert seen > 150
