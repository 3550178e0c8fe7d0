"""Operands of the panel kernel's matrix instructions are widened in an asm,
whose writes the compiler does not count when it places wait states: a matrix
instruction right behind one must still be two wait states away from it.
Compiles a few lines to gfx950 assembly and reads that; no GPU is involved."""

import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_28952_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "panel.h"
namespace pbs { namespace {
__global__ void probe(const float* a, const double* b, double* out) {
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b[threadIdx.x], widen_operand(a[threadIdx.x]), acc, 0, 0, 0);
  for (int i = 0; i < 4; ++i) out[4 * threadIdx.x + i] = acc[i];
}
}
void* probe_kernel() { return reinterpret_cast<void*>(probe); }
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no HIP compiler")
def test_widened_operand_keeps_its_distance(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text(SOURCE)
    out = tmp_path / "probe.s"
    cmd = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    code = [line.split(";")[0].strip() for line in out.read_text().splitlines()]
    code = [line for line in code if re.match(r"[vs]_", line) or line.startswith(("global_", "ds_", "buffer_"))]
    ends = [i for i, line in enumerate(code) if line.startswith("v_mfma_f64")]
    assert len(ends) == 1
    starts = [i for i, line in enumerate(code[:ends[0]]) if line.startswith("v_cvt_f64_f32")]
    assert starts
    states = 0
    for line in code[starts[-1] + 1:ends[0]]:
        nop = re.match(r"s_nop (\d+)", line)
        states += 1 + int(nop.group(1)) if nop else 1
    assert states >= 2, code[starts[-1]:ends[0] + 1]
