"""Compiled device code: the staged texture scatter adds through global atomics.  Its addresses pass through LDS as
integers; without their address space the compiler emits flat atomics, whose waits slow every kernel that holds one."""
import os
import subprocess

import pytest

HIPCC = "/opt/rocm/bin/hipcc"
CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2607_13265_amd", "csrc")
KERNEL = r"""
#include "ppt_device.h"
using namespace ppt;
template <int CH>
__global__ void k(double* a, const float* g) {
    __shared__ float stage[STAGE_WORDS];
    Bilin B;
    for (int q = 0; q < 4; ++q) { B.i[q] = q * CH; B.w[q] = g[q]; }
    scatter_staged<CH>(stage, a, B, g + 4, threadIdx.x & 1);
}
template __global__ void k<1>(double*, const float*);
template __global__ void k<3>(double*, const float*);
"""


def test_staged_scatter_has_no_flat_memory_instruction(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    from paper_2607_13265_amd import build
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(KERNEL)
    r = subprocess.run([HIPCC] + build.HIPCC_FLAGS + ["-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    ops = [line.split()[0] for line in asm.read_text().splitlines() if line.startswith("\t") and line.split()]
    assert sum(o.startswith("global_atomic_add_f64") for o in ops) == 2
    assert not [o for o in ops if o.startswith("flat_")]
