"""The launchers' slicing (a dispatch counts its threads in 32 bits), compiled
from the library's own sources for the CPU: every block and frame of a launch goes
out once, whatever the count, and S3 and S4 share a launch only while both fit
(test infrastructure; no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2505_01231_amd", "csrc")
EMU = os.path.join(HERE, "cpu_emulation")


def test_slices_cover_every_block_once(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    src = open(os.path.join(CSRC, "ps_fft.hip")).read()
    cut = re.search(r"\nhipError_t launch_dft\(", src)
    shift = re.search(r"\ntemplate <typename Args>\nvoid shift_classes\(.*?\n}\n", src, re.S)
    assert cut and shift, "launcher marker not found in ps_fft.hip"
    (tmp_path / "ps_fft_extract.inc").write_text(
        src[:cut.start()] + shift.group(0) + "\n}  // namespace\n}  // namespace ps\n")
    exe = tmp_path / "slices_driver"
    r = subprocess.run(["g++", "-std=c++20", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                        "-Wno-unknown-pragmas", "-Wno-unused-function", "-pthread", "-I", EMU, "-I", str(tmp_path),
                        "-I", CSRC, "-I", os.path.join(ROOT, "include"), os.path.join(EMU, "slices_driver.cpp"),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
