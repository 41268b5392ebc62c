"""The 16-byte stores written as asm end with the wait states that gfx950 asks
for before a vector write to a store's data registers: as many as the
compiler's own hazard pass puts there for the same store, which it does not see
in asm.  On the compiler's output, without a GPU."""
import os
import re
import subprocess

import pytest

from paper_2512_11473_amd import build

MIR = """---
name: f
tracksRegLiveness: true
body: |
  bb.0:
    liveins: $vgpr0_vgpr1, $vgpr2_vgpr3_vgpr4_vgpr5
    GLOBAL_STORE_DWORDX4 $vgpr0_vgpr1, $vgpr2_vgpr3_vgpr4_vgpr5, 0, 16, implicit $exec
    $vgpr2 = V_MOV_B32_e32 0, implicit $exec
    S_ENDPGM 0
...
"""

KERNEL = """
#include "common.hpp"
__global__ void stores(float *p, unsigned off, long long wide, float a) {
    const f32x4_t v = {a, a + 1, a + 2, a + 3};
    store_through(p, v);
    store_through(p, off, v * 2.0f);
    store_through(p, (int64_t)wide, v * 3.0f);
}
"""


def _after(lines, pattern):
    """Wait states of the s_nop that follows each match of the pattern."""
    got = []
    for i, line in enumerate(lines):
        if re.search(pattern, line):
            nop = re.match(r"s_nop (\d+)", lines[i + 1], re.IGNORECASE)
            got.append(int(nop.group(1)) + 1 if nop else 0)
    return got


def test_stores_keep_their_wait_states(tmp_path):
    llc = "/opt/rocm/llvm/bin/llc"
    if not (os.path.exists(build.HIPCC) and os.path.exists(llc)):
        pytest.skip("no compiler")
    mir, src = tmp_path / "store.mir", tmp_path / "stores.hip"
    mir.write_text(MIR)
    src.write_text(KERNEL)
    out = subprocess.run([llc, "-mtriple=amdgcn-amd-amdhsa", "-mcpu=gfx950", "-run-pass=post-RA-hazard-rec", str(mir),
                          "-o", "-"], capture_output=True, text=True, check=True).stdout
    wanted = _after([s.strip() for s in out.splitlines()], "GLOBAL_STORE_DWORDX4")
    assert wanted == [2]
    out = subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-device-only", "-S", str(src), "-o", "-"],
                         capture_output=True, text=True, check=True).stdout
    lines = [s.split(";")[0].strip() for s in out.splitlines()]
    got = _after([s for s in lines if s], r"global_store_dwordx4 .* sc1")
    assert len(got) == 3 and min(got) >= wanted[0], got
