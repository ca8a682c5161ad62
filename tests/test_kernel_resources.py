"""What the compiler gives the kernels that a caller's code or a large launch
depends on: registers spilled to memory, read from the code built here."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1408_6373_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# a function that holds three arrays of 16 words of a point
SOURCE = r"""
__device__ float ccuba_user(const float *x, int d, const float *a, const float *u) {
  float p[16], q[16], r[16], s = 0.0f;
  for (int j = 0; j < 16; ++j) {
    p[j] = j < d ? x[j] * a[j] : 0.0f;
    q[j] = p[j] * p[j] + (j < d ? u[j] : 0.0f);
    r[j] = sinf(q[j] - p[j]);
  }
  for (int j = 0; j < 16; ++j) s += p[j] * q[(j * 5 + 3) % 16] + r[(j * 3 + 1) % 16] * q[j];
  for (int j = 0; j < 16; ++j) s = s * 0.5f + r[j] * q[15 - j];
  return expf(-s * s);
}
"""


def _spills(asm):
    """{kernel symbol: vector registers spilled} of an assembly listing."""
    out = {}
    for part in asm.split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", part).group(1)
        out[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", part).group(1))
    return out


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_callers_integrands_do_not_spill(tmp_path):
    # the run-time compilation's own text and flags, compiled here
    src = tmp_path / "user.hip"
    inst = "".join(
        "template __global__ void ccuba::vegas_dosample_kernel<float, unsigned long long, 2, %d, "
        "true, true>(ccuba::VegasArgs);\n" % nb for nb in (2, 3, 4))
    src.write_text("#define CCUBA_RTC 1\n#include <hip/hip_runtime.h>\n" + SOURCE +
                   '#include "vegas_sample.h"\n' + inst)
    asm = tmp_path / "user.s"
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17",
                    "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I" + CSRC, "--cuda-device-only", "-S", str(src), "-o",
                    str(asm)], check=True, timeout=300)
    spills = _spills(asm.read_text())
    assert len(spills) == 3
    assert set(spills.values()) == {0}, spills
