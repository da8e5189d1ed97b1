"""A kernel that takes more than 64 KB of LDS is allowed to on every device it is launched on, and no later call takes that back. No GPU:
the few runtime functions that a launch needs are replaced by ones that keep a record, in a process of their own."""
import os
import subprocess
import sys

import pytest

from paper_2501_07145_amd import binding

RUNTIME = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
static int device, violations, launches, large, n;
static struct { int device; const void *kernel; int limit; } allowed[1024];
static struct { dim3 grid, block; size_t lds; void *stream; } pushed;
void test_set_device(int d) { device = d; }
int test_violations(void) { return violations; }
int test_launches(void) { return launches; }
int test_large(void) { return large; }
int hipGetDevice(int *d) { *d = device; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *kernel, int attribute, int value)
{
    (void)attribute;
    for (int i = 0; i < n; ++i)
        if (allowed[i].device == device && allowed[i].kernel == kernel) { allowed[i].limit = value; return 0; }
    allowed[n].device = device; allowed[n].kernel = kernel; allowed[n].limit = value;
    ++n;
    return value > 160 * 1024;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    (void)grid; (void)block; (void)args; (void)stream;
    ++launches;
    if (lds <= 64 * 1024) return 0;
    ++large;
    for (int i = 0; i < n; ++i)
        if (allowed[i].device == device && allowed[i].kernel == kernel && (size_t)allowed[i].limit >= lds) return 0;
    ++violations;
    return 0;
}
"""

CALLS = r"""
import ctypes, sys
runtime = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
class Shape(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int64), ("L", ctypes.c_int64), ("d", ctypes.c_int32), ("M", ctypes.c_int32), ("F", ctypes.c_int32),
                ("D", ctypes.c_int32), ("ld_out", ctypes.c_int64), ("rff_bf16", ctypes.c_int32), ("order", ctypes.c_int32)]
i64, i32, vp = ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p
lib.rfsf_ts_features.argtypes = [vp] * 5 + [ctypes.c_float, vp, vp, ctypes.c_size_t, vp]
lib.rfsf_dp1d_features.argtypes = [i64, i64, i32, i32, i32, vp, vp, vp, ctypes.c_float, vp, i64, vp]
NEVER_READ = 1 << 40
def ts(M, F, D):
    shape, size = Shape(300, 70, 12, M, F, D, 1 + M * D, 0, 1), ctypes.c_size_t()
    assert lib.rfsf_ts_workspace_bytes(ctypes.byref(shape), ctypes.byref(size), None) == 0
    p = NEVER_READ
    assert lib.rfsf_ts_features(ctypes.byref(shape), p, p, p, p, 1.0, p, p, size.value, None) == 0
def dp1d(M, F):
    p = NEVER_READ
    assert lib.rfsf_dp1d_features(4999, 257, 17, M, F, p, p, p, 1.0, p, 1 + M * F, None) == 0
def run():
    if sys.argv[3] == "dp1d":
        for M in (5, 2, 6): dp1d(M, 1000)
    elif sys.argv[3] == "tuned":
        for F in (700, 512, 1000): ts(5, F, 1024)
    elif sys.argv[3] == "wide":
        for F in (700, 512): ts(2, F, 4096)
    else:
        ts(9, 16, 4096)                      # nine levels: the general kernel
for device in (0, 3, 0, 1):
    runtime.test_set_device(device)
    run()
print(runtime.test_launches(), runtime.test_large(), runtime.test_violations())
"""


@pytest.mark.parametrize("kernels", ["dp1d", "tuned", "wide", "general"])
def test_every_device_allows_what_is_launched(tmp_path, kernels):
    source, runtime = tmp_path / "runtime.c", tmp_path / "libruntime.so"
    source.write_text(RUNTIME)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(runtime), str(source)], check=True)
    binding.load_library()
    env = dict(os.environ, HIP_VISIBLE_DEVICES="")
    out = subprocess.run([sys.executable, "-c", CALLS, str(runtime), binding.lib_path(), kernels], env=env, check=True,
                         capture_output=True, text=True).stdout.split()
    launches, large, violations = map(int, out[-3:])
    assert launches >= large >= 4 and violations == 0, out
