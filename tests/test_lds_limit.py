"""The coarse end of a multigrid cycle takes its LDS from a limit that belongs to
the kernel, shared by all threads: it is set to the largest coarse end's need and
never to a launch's own, so a small solve on one thread cannot lower it under a
large one on another.  On the CPU, with the runtime's calls recorded instead of
made."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_01735_amd", "librbgs.so")

RECORDER = r"""
#include <stddef.h>
#include <stdio.h>
typedef struct { unsigned x, y, z; } dim3;
static size_t pushed;
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void* f, int attr, int value) {
    printf("limit %d\n", value);
    return 0;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* s) { pushed = lds; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) {
    dim3 one = {1, 1, 1};
    *g = *b = one; *lds = pushed; *s = 0;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* s) {
    printf("launch %zu\n", lds);
    return 0;
}
"""

CALLS = r"""
import ctypes, sys
class Level(ctypes.Structure):
    _fields_ = [("u_red", ctypes.c_void_p), ("u_black", ctypes.c_void_p),
                ("f_red", ctypes.c_void_p), ("f_black", ctypes.c_void_p),
                ("pitch", ctypes.c_int64), ("n", ctypes.c_int),
                ("h2", ctypes.c_double), ("inv_h2", ctypes.c_double)]
class Levels(ctypes.Structure):
    _fields_ = [("level", Level * 8), ("count", ctypes.c_int), ("zero_top", ctypes.c_int)]
lib = ctypes.CDLL(sys.argv[1])
fn = lib["_ZN4rbgs23launch_mg_coarse_vcycleERKNS_14MgCoarseLevelsEiiiPKiP12ihipStream_t"]
for top in (15, 63, 7):
    lv = Levels()
    n = top
    while True:
        lv.level[lv.count].n = n
        lv.count += 1
        if n < 3:
            break
        n = (n - 1) // 2
    assert fn(ctypes.byref(lv), 1, 1, 1, None, None) == 0
"""


def test_limit_is_the_kernels_not_a_launchs(tmp_path):
    src, shim = tmp_path / "recorder.c", tmp_path / "recorder.so"
    src.write_text(RECORDER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(shim), str(src)], check=True)
    out = subprocess.run([sys.executable, "-c", CALLS, LIB], env={**os.environ, "LD_PRELOAD": str(shim)},
                         capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    events = [line.split() for line in out.stdout.splitlines()]
    launches = [int(v) for k, v in events if k == "launch"]
    assert len(launches) == 3 and launches[1] == max(launches)
    limit = 0
    for kind, value in events:
        if kind == "limit":
            assert int(value) >= limit, "a launch lowered the limit"
            limit = int(value)
            assert limit >= max(launches), "a limit too small for another thread's launch"
        else:
            assert int(value) <= limit
