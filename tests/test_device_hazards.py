"""Wait states that inline assembly has to spell out, read from the assembly that hipcc makes here.

gfx9 does not hold back a load to LDS that follows a scalar write of M0, its LDS address: one wait
state has to lie between them.  The compiler inserts it for its own builtins, not inside inline assembly.
"""
import os
import re
import subprocess

import pytest

from paper_2509_21009_amd import build

KERNEL = """
#include "lds_dma.hpp"
extern "C" __global__ void copies(const void* p, int a, int b, float* out) {
  __shared__ __attribute__((aligned(1024))) float s[4096];
  typedef const __attribute__((address_space(3))) char lds_char;
  const uint32_t lds = static_cast<uint32_t>((uintptr_t)(lds_char*)(s));
  const rollpack::u32x4_raw r = rollpack::raw_rsrc(p, 16384);
  rollpack::dma16(r, lds + a, threadIdx.x * 16);
  rollpack::dma16_nt(r, lds + b, threadIdx.x * 16);
  rollpack::wait_vmcnt<0>();
  __syncthreads();
  out[threadIdx.x] = s[threadIdx.x];
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_m0_wait_state_before_loads_to_lds(tmp_path):
    src = tmp_path / "copies.hip"
    src.write_text(KERNEL)
    asm = subprocess.run([build.HIPCC, *build.COMMON, *build.DEVICE, "--cuda-device-only", "-S", str(src), "-o", "-"],
                         check=True, capture_output=True, text=True, timeout=300).stdout
    code = [t for t in (ln.split(";")[0].strip() for ln in asm.splitlines()) if t and not t.startswith(".")]
    loads = [i for i, t in enumerate(code) if re.match(r"buffer_load_dwordx4 .*\blds$", t)]
    assert len(loads) == 2, code
    for i in loads:
        assert not re.match(r"s_\w+ m0,", code[i - 1]), code[i - 2:i + 1]
        assert any(re.match(r"s_\w+ m0,", t) for t in code[i - 3:i - 1]), code[i - 3:i + 1]


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_row_kernels_keep_their_partials_in_registers():
    """The row kernels load every split's partials before they add the first.  None spills, but for the
    residual norm of rows of more than 4,096 elements with 15 or 16 partials, which 128 registers do not hold."""
    asm = subprocess.run([build.HIPCC, *build.COMMON, *build.DEVICE, "--cuda-device-only", "-S",
                          os.path.join(build.CSRC, "k_elementwise.hip"), "-o", "-"],
                         check=True, capture_output=True, text=True, timeout=300).stdout
    scratch = {m.group(1): int(m.group(2)) for m in
               re.finditer(r"^(_Z\w+):.*?; ScratchSize: (\d+)", asm, flags=re.S | re.M)}
    assert any("k_rope_prefill" in k for k in scratch)
    spilled = {k for k, v in scratch.items() if v > 0}
    wide = {k for k in scratch if re.search(r"k_add_rmsnormI[tf]Li1[56]ELi1024E", k)}
    assert len(wide) == 4 and spilled <= wide, spilled - wide
