"""The rules of csrc/launch_rules.hpp at their lines, in a small host program."""
import os
import shutil
import subprocess

import pytest

from paper_2509_17257_amd import build as hip_build

PROGRAM = r"""
#include "launch_rules.hpp"
int main() {
    using h2x::leaf_two_waves;
    if (!leaf_two_waves(2048, 33, 30000) || !leaf_two_waves(100000, 64, 36000)) return 1;
    if (leaf_two_waves(2047, 64, 30000)) return 2;   // fewer than twice the chip
    if (leaf_two_waves(100000, 32, 1000)) return 3;  // at most two row tiles
    // a table of near rows that leaves room for three or two work-groups on a CU
    if (leaf_two_waves(100000, 64, 4 * 10730) || leaf_two_waves(100000, 100, 4 * 13905)) return 4;
    // FP32 and BF16: one round of two-wave groups, or more than two and a half times the chip
    using h2x::leaf_two_waves_lp;
    if (!leaf_two_waves_lp(1280, 2, 64, 8000) || !leaf_two_waves_lp(1536, 1, 64, 16384)) return 5;
    if (leaf_two_waves_lp(1279, 2, 64, 8000) || leaf_two_waves_lp(1537, 2, 64, 8000)) return 6;
    if (leaf_two_waves_lp(1400, 2, 64, 16385) || leaf_two_waves_lp(1400, 2, 32, 8000) || leaf_two_waves_lp(1400, 2, 65, 8000)) return 7;
    if (leaf_two_waves_lp(2559, 2, 64, 8000) || !leaf_two_waves_lp(2560, 2, 64, 8000)) return 8;
    if (!leaf_two_waves_lp(2048, 3, 64, 8000) || leaf_two_waves_lp(1400, 3, 64, 8000)) return 9;
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_leaf_two_waves(tmp_path):
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{hip_build.CSRC}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
