"""Values handed from lane to lane of one wave through LDS (the small-rank FP64 coupling): on every
path of the compiled kernel a wave barrier, which the compiler moves no memory operation across,
or a work-group barrier stands between LDS stores and the LDS loads that follow them, and between
loads and the stores that follow.  Checked in the device code's intermediate form (host only)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_17257_amd import build as hip_build

SOURCE = r"""
#include "coupling_small.hpp"
namespace h2x {
#define K(P, NJ, SP)                                                                                        \
    template __global__ void k_coupling_small<P, NJ, SP>(int64_t, int32_t, int32_t, const int32_t *,        \
        const int64_t *, const int32_t *, const double *, const double *, double *, int64_t, Skip, int);
K(1, 1, 1) K(1, 2, 1) K(1, 1, 4) K(1, 2, 4) K(2, 1, 1) K(2, 2, 1) K(2, 1, 4) K(2, 2, 4) K(3, 1, 4) K(3, 2, 4)
}
"""


def _blocks(body):
    """label -> (lines, successors) of a function's text"""
    blocks, cur = {}, []
    label = "entry"
    for line in body.splitlines():
        m = re.match(r"^([\w.$-]+):", line)
        if m:
            blocks[label], cur, label = cur, [], m.group(1)
        else:
            cur.append(line.strip())
    blocks[label] = cur
    return {k: (v, [s for l in v if re.match(r"(br|switch|\]|i32 \d+, label)", l)
                    for s in re.findall(r"label %([\w.$-]+)", l)]) for k, v in blocks.items()}


def _unordered(body):
    """LDS accesses that follow one of the other kind without a barrier between, over all paths"""
    blocks = _blocks(body)
    first = next(iter(blocks))
    seen, todo, bad, lds = set(), [(first, "")], set(), 0
    while todo:
        label, last = todo.pop()
        if (label, last) in seen:
            continue
        seen.add((label, last))
        lines, succ = blocks[label]
        for line in lines:
            if "llvm.amdgcn.wave.barrier" in line or "llvm.amdgcn.s.barrier" in line:
                last = ""
            elif re.search(r"^store .*addrspace\(3\)|= load .*addrspace\(3\)", line):
                kind = "store" if line.startswith("store") else "load"
                lds += 1
                if last and last != kind:
                    bad.add((label, line))
                last = kind
        todo += [(s, last) for s in succ]
    return bad, lds


@pytest.mark.skipif(not os.path.exists(hip_build.HIPCC) and shutil.which("hipcc") is None, reason="no hipcc")
def test_small_coupling(tmp_path):
    src, out = tmp_path / "k.hip", tmp_path / "k.ll"
    src.write_text(SOURCE)
    flags = [f for f in hip_build.HIP_FLAGS if f != "-Wall"]
    subprocess.run([hip_build.HIPCC, *flags, f"-I{hip_build.CSRC}", "--cuda-device-only", "-S", "-emit-llvm", str(src),
                    "-o", str(out)], check=True, capture_output=True, timeout=600)
    kernels = re.findall(r"define[^\n]*amdgpu_kernel void @(\w*k_coupling_small\w*)\([^\n]*\{\n(.*?)\n\}", out.read_text(),
                         re.S)
    assert len(kernels) == 10
    for name, body in kernels:
        bad, lds = _unordered(body)
        assert lds > 0, name
        assert not bad, (name, sorted(bad)[:3])
