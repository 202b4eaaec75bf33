"""Exchanges between the lanes of one wave through LDS have no workgroup barrier; what
keeps their writes and reads apart is a wave barrier, checked here in the compiler's
intermediate code (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2601_04904_amd import build

KERNEL = """
#include "tile16.h"
using namespace btsq;
__global__ void turned(double2* x) {
    __shared__ Turn X;
    double2 v[4];
    for (int t = 0; t < 4; ++t) v[t] = x[64 * t + threadIdx.x];
    turn16(v, X, threadIdx.x & 15, threadIdx.x >> 4);
    for (int t = 0; t < 4; ++t) x[64 * t + threadIdx.x] = v[t];
}
__global__ void rows(double2* x, const int* piv) {
    __shared__ SmallInvLds<1, 1> L;
    DevStatus* none = nullptr;
    small_inverse<1, 1>(x, x, 16, 0, L, threadIdx.x, none);
}
"""


@pytest.fixture(scope="module")
def ir(tmp_path_factory):
    if shutil.which(build.HIPCC) is None:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("ir")
    src, out = d / "k.hip", d / "k.ll"
    src.write_text(KERNEL)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([build.HIPCC, "-w"] + flags + ["-I", build.CSRC, "--offload-device-only", "-S", "-emit-llvm",
                                                  str(src), "-o", str(out)], check=True)
    return out.read_text()


def events(ir, name):
    """The LDS writes (W), LDS reads (R) and wave or workgroup barriers (|) of a kernel, in order."""
    body = re.search(r"define[^\n]*@_Z\d+%s\w*\(.*?\n}" % name, ir, re.S).group(0)
    seq = ""
    for line in body.splitlines():
        if re.search(r"\bstore\b.*addrspace\(3\)|llvm\.memcpy\.p3\.", line):
            seq += "W"
        elif re.search(r"= load\b.*addrspace\(3\)|llvm\.memcpy\.p\d\.p3\.", line):
            seq += "R"
        elif "amdgcn.wave.barrier" in line or "amdgcn.s.barrier" in line:
            seq += "|"
    return seq


def test_turned_operands(ir):
    assert re.fullmatch(r"W+\|R+\|", events(ir, "turned"))


def test_pivot_rows_of_the_small_inverse(ir):
    """Reads of the pivot rows (the read after the conditional writes of four row blocks) never
    follow a write without a barrier."""
    seq = events(ir, "rows")
    assert "W" in seq and "R" in seq
    assert "WR" not in seq, seq
