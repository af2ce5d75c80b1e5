"""copy_to_lds tells the compiler that it writes the register of LDS addresses, m0: a builtin that needs another address
behind it gets its own again.  Read off the assembly of a small kernel; no GPU is needed."""
import re
import subprocess

from paper_2408_02937_amd import build

KERNEL = r"""
#include "rtams_dev.h"
using namespace rtams;
typedef __attribute__((address_space(1))) const void Global;
typedef __attribute__((address_space(3))) void Lds;
__global__ void k(const float *a, const float *b, float *out) {
  __shared__ __attribute__((aligned(1024))) float lds[1024];
  Lds *to = (Lds *)lds;
  __builtin_amdgcn_global_load_lds((Global *)(a + threadIdx.x), to, 4, 0, 0);
  copy_to_lds(b, lds_address(lds) + 2048, threadIdx.x * 16u);
  __builtin_amdgcn_global_load_lds((Global *)(a + 64 + threadIdx.x), to, 4, 256, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  out[threadIdx.x] = lds[threadIdx.x * 5 % 1024];
}
"""


def test_the_address_register_is_set_again_behind_a_copy(tmp_path):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(KERNEL)
    subprocess.run(["/opt/rocm/bin/hipcc", *build.FLAGS, "--offload-device-only", "-S", "-I", build.CSRC, str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    steps = re.findall(r"^\s*(global_load_lds_\w+|s_mov\w*_b32 m0|s_movk_i32 m0)", asm.read_text(), re.M)
    kinds = ["m0" if "m0" in s else "copy" if s.endswith("x4") else "builtin" for s in steps]
    assert kinds == ["m0", "builtin", "m0", "copy", "m0", "builtin"], kinds
