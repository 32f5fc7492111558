"""load_lds16 (fa_common.h) takes its place in LDS from m0, where code that the
compiler generates around it may hold a value (no GPU).  A kernel whose own load
to LDS stands before and after one: m0 must be written again for the second."""
import subprocess

from paper_2608_18656_amd import build as hip_build

KERNEL = r"""
#include "fa_common.h"
typedef __attribute__((address_space(3))) void lds_void;
__global__ void probe(const char *a, const char *b, float *o) {
    __shared__ float s[1024];
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(a), (short)0, 4096, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)s, 4, 4 * threadIdx.x, 0, 0, 0);
    fa::load_lds16(b, 4096, fa::lds_address(s + 512), 16 * threadIdx.x);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)s, 4, 4 * threadIdx.x, 0, 1024, 0);
    fa::lds_loads_done<0>();
    __syncthreads();
    o[threadIdx.x] = s[threadIdx.x] + s[threadIdx.x + 512];
}
"""


def test_m0_is_known_to_change(tmp_path):
    src, out = tmp_path / "p.hip", tmp_path / "p.s"
    src.write_text(KERNEL)
    subprocess.run([hip_build.hipcc(), *hip_build.HIPCC_FLAGS, "-w", "-I", hip_build.CSRC, "--cuda-device-only", "-S",
                    str(src), "-o", str(out)], check=True, capture_output=True)
    text = out.read_text()
    before, after = text.split("probe", 1)[1].split("#ASMSTART", 1)[0], text.split("#ASMEND", 1)[1]
    assert "lds" in before and "m0" in before   # the first load sets m0
    second = after.split("buffer_load_dword ", 1)
    assert len(second) == 2, "no load after the block"
    assert "s_mov_b32 m0" in second[0] or "m0," in second[0]
