"""The written-out integer inner loop (update4) as the compiler allocates it: a
cell's minimum is written before later cells read their operands, so no operand
may share a register with a cell, whatever values they are known to share.  The
block is compiled for gfx950 with every operand the same value, the case in
which the compiler would share registers if it may, and its register use read
from the assembly."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "fw_tiles.h"
template <class A>
__device__ void go(const int *in, int *out) {
    const int v = in[threadIdx.x];
    int c[4] = {v, v, v, v}, b0[4] = {v, v, v, v}, b1[4] = {v, v, v, v};
    fw::update4<A>(c, v, v, b0, b1);
    for (int e = 0; e < 4; ++e) out[threadIdx.x * 4 + e] = c[e];
}
extern "C" __global__ void plain(const int *in, int *out) { go<fw::Ar<int32_t>>(in, out); }
extern "C" __global__ void keyed(const int *in, int *out) { go<fw::ArKey>(in, out); }
"""


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if shutil.which(HIPCC) is None:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("update4")
    src, out = d / "u.hip", d / "u.s"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "-x", "hip", "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "paper_1001_4108_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"), "-S", "--offload-device-only",
                    str(src), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


@pytest.mark.parametrize("kernel", ["plain", "keyed"])
def test_no_operand_is_overwritten_before_its_use(assembly, kernel):
    body = assembly[assembly.index(f"\n{kernel}:"):]
    block = body[body.index("ASMSTART"):body.index("ASMEND")]
    cells, sums = set(), set()
    minima = 0
    for op, regs in re.findall(r"^\s*(v_\w+)\s+(.*)$", block, re.M):
        dst, *srcs = [r.strip() for r in regs.split(",")]
        if op == "v_add_u32":
            # its operands are the caller's values, never a result of this block
            assert not set(srcs) & (cells | sums), (op, regs)
            sums.add(dst)
        else:
            assert op == "v_min3_i32" and srcs[0] == dst and set(srcs[1:]) <= sums, (op, regs)
            assert dst not in cells | sums
            cells.add(dst)
            minima += 1
    assert minima == 4
