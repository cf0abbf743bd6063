"""Device code that only the compiler's output can check: compiled for gfx950 here, no GPU needed."""
import re
import shutil
import subprocess

import pytest

from paper_2605_10380_amd import build as X

PROBE = r"""
#include <hip/hip_runtime.h>
#include "lds_copy.h"
typedef const __attribute__((address_space(1))) void* global_ptr;
typedef __attribute__((address_space(3))) void* lds_ptr;
__global__ void probe(const float* a, const char* b, float* out) {
    __shared__ __attribute__((aligned(1024))) char s[2048];
    auto* lds = (__attribute__((address_space(3))) char*)s;
    __builtin_amdgcn_global_load_lds((global_ptr)(a + threadIdx.x), (lds_ptr)lds, 4, 0, 0);
    ax::copy_to_lds(b, threadIdx.x * 16, (unsigned)(size_t)lds + 1024);
    __builtin_amdgcn_global_load_lds((global_ptr)(a + 64 + threadIdx.x), (lds_ptr)lds, 4, 0, 0);
    ax::wait_copies_and_sync<0>();
    out[threadIdx.x] = ((float*)s)[threadIdx.x];
}
"""


@pytest.mark.skipif(not shutil.which(X.HIPCC), reason="no hipcc")
def test_copy_to_lds_tells_the_compiler_about_m0(tmp_path):
    """The copy needs m0, the LDS address of such a load.  A load of the compiler's own before and one behind it, at the same LDS
    address: the second may not rely on the m0 of the first."""
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    r = subprocess.run([X.HIPCC, *X.FLAGS, "-I", X.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    seq = re.findall(r"^\s*(s_\w+ m0|global_load_lds_dword\w*)", out.read_text(), flags=re.M)
    loads = [i for i, x in enumerate(seq) if x.startswith("global_load_lds")]
    assert [seq[i] for i in loads] == ["global_load_lds_dword", "global_load_lds_dwordx4", "global_load_lds_dword"]
    assert all("m0" in seq[i - 1] for i in loads), seq
