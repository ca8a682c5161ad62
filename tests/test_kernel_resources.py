"""What the compiler gives the kernels that a caller's code or a large launch
depends on: registers spilled to memory, read from the code built here."""
import os
import re
import subprocess

import pytest

import paper_1408_6373_amd as cc

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1408_6373_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LLVM = "/opt/rocm/llvm/bin"

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


def _library_scratch(tmp_path):
    """{kernel symbol: bytes of scratch a lane} of the built library."""
    fat = tmp_path / "fatbin"
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=%s" % fat,
                    cc._lib._name, str(tmp_path / "stripped")], check=True, timeout=60)
    data = fat.read_bytes()
    at = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)] + [len(data)]
    out = {}
    for q in range(len(at) - 1):
        bundle, code = tmp_path / ("b%d" % q), tmp_path / ("b%d.co" % q)
        bundle.write_bytes(data[at[q]:at[q + 1]])
        subprocess.run([LLVM + "/clang-offload-bundler", "--type=o", "--unbundle",
                        "--input=%s" % bundle, "--output=%s" % code,
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True, timeout=60)
        notes = subprocess.run([LLVM + "/llvm-readobj", "--notes", str(code)], check=True,
                               capture_output=True, text=True, timeout=60).stdout
        for part in re.split(r"- \.agpr_count:", notes)[1:]:
            name = re.search(r"\.symbol:\s+'?(\S+?)\.kd'?\n", part).group(1)
            out[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", part).group(1))
    return out


@pytest.mark.skipif(not os.path.exists(LLVM + "/clang-offload-bundler"), reason="needs LLVM tools")
def test_cuhre_lane_rules_use_no_scratch(tmp_path):
    # the rule launches of 512 regions and more at up to 8 dimensions
    scratch = {k: v for k, v in _library_scratch(tmp_path).items() if "gm_rule_lane" in k}
    assert len(scratch) >= 5 * 7  # every family and dimension
    assert set(scratch.values()) == {0}, scratch
