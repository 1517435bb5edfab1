"""The assembly transfer of tmla_lds_asm.hpp sets M0 itself.  The compiler has to know, or a transfer of its
own builtin behind it, whose M0 it believes to be set already, lands where the assembly one went."""
import os
import re
import subprocess

import pytest

from paper_2509_21081_amd import build as B

PROBE = r'''
#include "%s/tmla_lds_asm.hpp"
using namespace tmla;
__global__ void m0_probe(const char* src, float* out) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  dma16(src + threadIdx.x * 16, smem);
  dma16_scalar_base<false>(threadIdx.x * 16, src, lds_addr(smem), 4096);
  dma16_scalar_base<true>(threadIdx.x * 16, src, lds_addr(smem), 8192);
  dma16(src + 1024 + threadIdx.x * 16, smem);
  vm_wait<0>();
  raw_barrier();
  out[threadIdx.x] = lds_read_f32_now(lds_addr(smem) + threadIdx.x * 4);
}
'''


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_a_builtin_transfer_behind_an_assembly_one_has_its_own_m0(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text(PROBE % B.CSRC)
    out = tmp_path / "probe.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "-S", "--cuda-device-only", "-o", str(out), str(src)], check=True,
                   capture_output=True)
    text = out.read_text()
    body = text[text.index("m0_probe"):text.index(".Lfunc_end")]
    writer, seen = None, []
    for line in body.split("\n"):
        if re.match(r"\s*s_\w+ m0,", line):
            writer = line.strip()
        elif "global_load_lds" in line:
            seen.append(writer)
    assert len(seen) == 4
    # the second builtin transfer goes to the start of the LDS, not to the assembly transfers' places
    assert "s_add_u32" in seen[1] and "s_add_u32" in seen[2] and "s_add_u32" not in seen[3], seen
