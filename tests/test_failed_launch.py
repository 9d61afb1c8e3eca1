"""What a step leaves behind when one of its launches fails, for every launch of it: no GPU, a stand-in takes the runtime's launch calls."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# Loaded before the library, so that the library's calls end here.  The launch numbered `fail_at` returns an error.
STAND_IN = r"""
#include <hip/hip_runtime.h>
extern "C" {
static int launches = 0, fail_at = -1;
static hipError_t last = hipSuccess;
void stand_in_reset(int at) { launches = 0; fail_at = at; last = hipSuccess; }
int stand_in_launches() { return launches; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  last = launches++ == fail_at ? hipErrorLaunchFailure : hipSuccess;
  return last;
}
hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { p->multiProcessorCount = 256; return hipSuccess; }
}
"""

# Addresses are never read: nothing runs.
PROGRAM = r"""
import ctypes as C, sys
stand_in = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2403_04865_amd import binding as B
lib = B.load_cdll()
N, CHUNK = 10, 4
cfg = B._CConfig(32, 8, 64, 2, 2, 4, 32, 1, int(sys.argv[3]), int(sys.argv[4]), 1e-6, 0)
ctx = C.c_void_p()
assert lib.slide_ctx_create(C.byref(cfg), C.byref(ctx)) == 0
size = max(lib.slide_chunked_arena_bytes(ctx, N, CHUNK), lib.slide_arena_bytes(ctx, N))
at = [C.c_void_p(0x10000000 + 0x10000000 * i) for i in range(8)]
assert lib.slide_bind(ctx, at[0], at[1], at[2], size) == 0
def chunked(): return lib.slide_step_chunked(ctx, at[3], N, CHUNK, 0, 0, at[4], at[5], at[6], at[7], None)
def whole(): return lib.slide_step_fwd(ctx, at[3], N, 0, at[4], at[5], at[6], None)
for step, tiles in ((chunked, (CHUNK, N % CHUNK)), (whole, (N,))):
    stand_in.stand_in_reset(-1)
    assert step() == 0
    total = stand_in.stand_in_launches()
    assert total > 20
    for k in range(total):
        stand_in.stand_in_reset(k)
        assert step() == -5, (step.__name__, k)                                           # SLIDE_EHIP
        stand_in.stand_in_reset(-1)
        for n in tiles:
            rc = lib.encoder_bwd_tiles(ctx, at[7], n, 0, None, None)
            assert rc == -4, (step.__name__, k, n, rc)                                    # SLIDE_ESTATE
        assert lib.slide_step_bwd(ctx, 0, None, None) == -4, (step.__name__, k)
        assert stand_in.stand_in_launches() == 0
    print(step.__name__, total, "launches")
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    from paper_2403_04865_amd.binding import lib_path
    from paper_2403_04865_amd.build import _hipcc, build
    if not os.path.exists(lib_path()):
        build()
    d = tmp_path_factory.mktemp("stand_in")
    (d / "stand_in.hip").write_text(STAND_IN)
    (d / "program.py").write_text(PROGRAM)
    subprocess.run([_hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "stand_in.hip"), "-o", str(d / "stand_in.so"),
                    "-no-hip-rt"], check=True, capture_output=True)
    return d


@pytest.mark.parametrize("dtype,recompute", [(0, 0), (1, 0), (1, 1)])
def test_no_backward_on_a_failed_step(stand_in, dtype, recompute):
    p = subprocess.run([sys.executable, str(stand_in / "program.py"), str(stand_in / "stand_in.so"), ROOT, str(dtype), str(recompute)],
                       capture_output=True, text=True, timeout=100)
    print(p.stdout, p.stderr)
    assert p.returncode == 0
