"""Kernels whose result must not depend on the order in which a block's threads
run between two barriers, run on the CPU in both orders (tests/cpu)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2112_00087_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.parametrize("source,end,define", [("bicgstabl.hip", "template <typename T, int LL>\nint enqueue_mr", "BICGSTABL"),
                                               ("tfqmr.hip", "}  // namespace\n\ntemplate <typename T>\nint tfqmr_run", "TFQMR")])
def test_settle_does_not_depend_on_thread_order(tmp_path, source, end, define):
    with open(os.path.join(CSRC, source)) as fh:
        text = fh.read()
    assert text.count(end) == 1
    part = tmp_path / "device_part.h"
    part.write_text(text[:text.index(end)] + "\n}  // namespace\n")
    with open(os.path.join(CSRC, "ops.h")) as fh:      # its launches are calls on the CPU
        (tmp_path / "ops.h").write_text(re.sub(r"<<<.*?>>>", "", fh.read(), flags=re.S))
    exe = tmp_path / "settle"
    cmd = [CLANG, "-std=c++17", "-O1", "-w", f"-D{define}", f'-DDEVICE_PART="{part}"',
           "-I" + os.path.join(ROOT, "tests", "cpu"), "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
           "-I/opt/rocm/include", os.path.join(ROOT, "tests", "cpu", "settle.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
