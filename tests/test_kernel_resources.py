"""The leaf stage's kernels hold their operands in registers: none of them uses scratch memory (host
only, from the compiler's resource lines)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_17257_amd import build as hip_build


@pytest.mark.skipif(not os.path.exists(hip_build.HIPCC) and shutil.which("hipcc") is None, reason="no hipcc")
def test_leaf_kernels_use_no_scratch(tmp_path):
    out = tmp_path / "matmul.s"
    flags = [f for f in hip_build.HIP_FLAGS if f != "-Wall"]
    subprocess.run([hip_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(hip_build.CSRC, "matmul.hip"), "-o",
                    str(out)], check=True, capture_output=True, timeout=900)
    used = {m.group(1): int(m.group(2))
            for m in re.finditer(r"\.amdhsa_kernel (\S*k_leaf_cat\S*)\n.*?private_segment_fixed_size (\d+)",
                                 out.read_text(), re.S)}
    assert len(used) >= 20
    assert not {k: v for k, v in used.items() if v}
