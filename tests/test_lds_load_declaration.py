"""The inline assembly that loads from memory straight to LDS declares what it changes besides its operands:
M0 and memory.  Looked up in the compiler's intermediate code of a kernel of its own."""
import os
import re
import subprocess

from paper_2602_12128_amd import build

KERNEL = """
#include "hla_handle.h"
#include "hla_mfma_common.h"
__global__ void probe(const uint32_t* src, uint32_t* out) {
  __shared__ __align__(16) unsigned char buf[1024];
  hla::mf::load_to_lds16(src + 4 * threadIdx.x, buf);
  hla::mf::wait_lds_loads();
  __syncthreads();
  out[threadIdx.x] = reinterpret_cast<const uint32_t*>(buf)[threadIdx.x];
}
"""


def test_load_to_lds_declares_m0_and_memory(tmp_path):
    src, ir = str(tmp_path / "probe.hip"), str(tmp_path / "probe.ll")
    with open(src, "w") as f:
        f.write(KERNEL)
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", src, "-o", ir], check=True,
                   capture_output=True)
    calls = [line for line in open(ir) if "global_load_lds_dwordx4" in line and " asm " in line]
    assert calls
    for line in calls:
        changed = set(re.findall(r"[~=]\{(\w+)\}", line))  # outputs and clobbers
        assert {"m0", "memory"} <= changed, line
        assert "sideeffect" in line
