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
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_leaf_two_waves(tmp_path):
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{hip_build.CSRC}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
