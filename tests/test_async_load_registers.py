"""The asynchronous loads to LDS (pat_dev.h) set m0, where the compiler keeps the LDS base of loads to LDS that it issues
itself: it has to set it anew after them.  Read from the assembly of a small kernel compiled here; needs no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

KERNEL = r"""
#include "pat_dev.h"
typedef __attribute__((address_space(3))) void *lds_t;
typedef const __attribute__((address_space(1))) void *mem_t;
__global__ void between(const char *a, const char *b, float *out)
{
    __shared__ __align__(16) char buf[4096];
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_global_load_lds((mem_t)(a + lane * 16), (lds_t)buf, 16, 0, 0);
    pat::%s(b, lane * 16, pat::lds_offset(buf) + 1024);
    __builtin_amdgcn_global_load_lds((mem_t)(a + 4096 + lane * 16), (lds_t)buf, 16, 0, 0);
    __syncthreads();
    out[threadIdx.x] = reinterpret_cast<float *>(buf)[threadIdx.x];
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("load", ["load_to_lds", "load_to_lds_stream"])
def test_m0_is_set_anew_after_an_asynchronous_load(load, tmp_path):
    src = tmp_path / "between.hip"
    src.write_text(KERNEL % load)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2605_23945_amd", "csrc"),
                        "--cuda-device-only", "-S", "-o", "-", str(src)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "warning: inline asm" not in r.stderr
    lines = [l.strip() for l in r.stdout.splitlines()]
    loads = [i for i, l in enumerate(lines) if l.startswith("global_load_lds_dwordx4")]
    sets = [i for i, l in enumerate(lines) if l.startswith("s_mov_b32 m0") or (l.startswith("s_") and " m0," in l)]
    assert len(loads) == 3
    for prev, at in zip([-1] + loads, loads):                  # each load has its own base, set after the load before it
        assert any(prev < s < at for s in sets), "\n".join(lines[max(prev, 0):at + 1])
