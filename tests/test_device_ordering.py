"""What the compiler is told about a wavefront's exchanges through LDS: a lane reads what other lanes of its wavefront wrote, which only a fence
says.  Compiled here to LLVM IR; no GPU involved."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_14638_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
EXCHANGE = """
#include "linear_epilogue.hpp"
using namespace w4a8;
extern "C" __global__ void __launch_bounds__(64) exchange(const v4f* sums, TYPE* y, int M, int N, int64_t ldy, float scale) {
    __shared__ __attribute__((aligned(16))) uint8_t slab[OutLayout<TYPE, 2>::SLAB_BYTES];
    v4f acc[4][2];
    for (int f = 0; f < 4; ++f)
        for (int j = 0; j < 2; ++j) acc[f][j] = sums[(f * 2 + j) * 64 + threadIdx.x];
    store_tile<TYPE, 4, 2, false, 0, 4>(acc, slab, 0, 0, M, N, y, ldy, scale, nullptr, 0, StaticQuantizer(scale), threadIdx.x);
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("kind", ["float", "uint16_t", "uint8_t", "SiluFp8"])
def test_epilogue_rounds_are_fenced(tmp_path, kind):
    """Before each round's writes to the slab and between them and the reads."""
    source, ir = str(tmp_path / "exchange.hip"), str(tmp_path / "exchange.ll")
    with open(source, "w") as f:
        f.write(EXCHANGE.replace("TYPE", kind))
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", CSRC, "--cuda-device-only", "-S", "-emit-llvm", source, "-o", ir]
    done = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert done.returncode == 0, done.stdout[-4000:]
    rounds, open_writes, fences = 0, False, 0
    for line in open(ir):
        if "addrspace(3)" in line and line.lstrip().startswith("store"):
            assert fences > 0 or open_writes, "written over what may still be read"
            open_writes, fences = True, 0
        elif "addrspace(3)" in line and " = load " in line:
            assert not open_writes, "read before a fence"
        elif 'fence syncscope("wavefront") acq_rel' in line:
            rounds += open_writes
            open_writes, fences = False, fences + 1
    assert rounds >= 1
