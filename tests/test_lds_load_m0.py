"""load_to_lds (csrc/device_common.h) writes m0 in inline asm: a builtin load to
LDS behind it has to set m0 again, read from the generated gfx950 assembly."""
import os
import re
import subprocess

import pytest

from paper_2605_20600_amd.build import CSRC, HIPCC_FLAGS, hipcc

KERNEL = """
#include <hip/hip_runtime.h>
#include "device_common.h"
using namespace headkv::dev;
typedef __attribute__((address_space(1))) const unsigned g_t;
typedef __attribute__((address_space(3))) unsigned l_t;
__global__ void k(const uint16_t* a, const unsigned* b, unsigned* out, uint32_t where) {
    extern __shared__ unsigned lds[];
    __builtin_amdgcn_global_load_lds((g_t*)b, (l_t*)lds, 4, 0, 0);
    load_to_lds<ONCE>(a + 8 * threadIdx.x, where);
    __builtin_amdgcn_global_load_lds((g_t*)(b + 64), (l_t*)lds, 4, 0, 0);
    lds_loads_done();
    __syncthreads();
    out[threadIdx.x] = lds[threadIdx.x];
}
"""


@pytest.mark.parametrize("once", ["false", "true"])
def test_m0_is_set_again_behind_the_asm_load(once, tmp_path):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(KERNEL.replace("ONCE", once))
    subprocess.run([hipcc(), *HIPCC_FLAGS, "-I", CSRC, "--cuda-device-only", "-S", str(src),
                    "-o", str(asm)], check=True, capture_output=True,
                   env={**os.environ, "TMPDIR": str(tmp_path)})
    ops = re.findall(r"^\s*(s_mov_b32 m0|global_load_lds_\w+)", asm.read_text(), re.M)
    behind = ops[ops.index("global_load_lds_dwordx4") + 1:]
    assert behind == ["s_mov_b32 m0", "global_load_lds_dword"], ops
