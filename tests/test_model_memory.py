"""Creating a model where memory is short: the buffers that a model needs come
first, and the Jacobian's tapes, which it can do without, take what is left.
The library is loaded in a process of its own over stand-ins for the device
calls it makes (an allocator of a given number of bytes; copies and launches
do nothing), so no device is needed."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_18065_amd", "libminsr.so")

STAND_INS = r"""
#include <stddef.h>
static size_t limit, used, count, at[4096][2];
void set_limit(size_t b) { limit = b; }
size_t in_use(void) { return used; }
int hipMalloc(void** p, size_t n) {
  if (n > limit - used || count == 4096) { *p = 0; return 2; }
  used += n;
  at[count][0] = 4096 * (count + 1); at[count][1] = n;
  *p = (void*)at[count++][0];
  return 0;
}
int hipFree(void* p) {
  for (size_t i = 0; i < count; ++i)
    if (at[i][0] == (size_t)p) { used -= at[i][1]; at[i][1] = 0; at[i][0] = 0; }
  if (used == 0) count = 0;
  return 0;
}
int hipMemGetInfo(size_t* f, size_t* t) { *f = limit - used; *t = limit; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { return 0; }
int hipMemset(void* d, int v, size_t n) { return 0; }
int hipGetLastError(void) { return 0; }
typedef struct { unsigned x, y, z; } dim3_;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t m, void* s) { return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* m, void** s) { return 0; }
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** a, size_t m, void* s) { return 0; }
"""

# prints the bytes a model holds with memory to spare, the least memory that
# creates it, and of 40 amounts in between those that do not
SCRIPT = r"""
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
shim.set_limit.argtypes = [C.c_size_t]; shim.in_use.restype = C.c_size_t
class Desc(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("Lx", "Ly", "dim", "hidden", "cplx", "marshall", "zm", "dt")] + [
        ("seed", C.c_uint64), ("max_Ns", C.c_int32), ("options", C.c_int32)]
d = Desc(*[int(v) for v in sys.argv[3:14]])
lib.minsr_destroy_model.argtypes = [C.c_void_p]
def held(limit):
    shim.set_limit(limit)
    h = C.c_void_p()
    rc = lib.minsr_create_model(C.byref(d), C.byref(h))
    n = shim.in_use()
    if rc == 0:
        lib.minsr_destroy_model(h)
    assert shim.in_use() == 0
    return n if rc == 0 else -1
most = held(1 << 40)
lo, hi = 0, 1 << 40
while hi - lo > 1:
    mid = (lo + hi) // 2
    lo, hi = (lo, mid) if held(mid) >= 0 else (mid, hi)
least = hi
print(most, least, *[b for b in (least + (most - least) * k // 40 for k in range(41)) if held(b) < 0])
"""


@pytest.mark.skipif(not os.path.exists(LIB) or not shutil.which("gcc"), reason="library or gcc missing")
@pytest.mark.parametrize("desc", [
    (10, 10, 2, 128, 0, 1, 1, 1, 1, 4096, 0), (6, 6, 2, 32, 1, 1, 0, 0, 1, 251, 0),
    (40, 1, 1, 64, 1, 0, 0, 0, 1, 2048, 1), (9, 1, 1, 8, 0, 0, 0, 0, 1, 5, 0),
])
def test_creation_needs_no_memory_for_the_tapes(tmp_path, desc):
    import paper_2608_18065_amd as pm
    desc = desc[:7] + ((pm.F64, pm.F32)[desc[7]],) + desc[8:]
    (tmp_path / "s.c").write_text(STAND_INS)
    so = str(tmp_path / "s.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", so, str(tmp_path / "s.c")], check=True)
    r = subprocess.run([sys.executable, "-c", SCRIPT, so, LIB] + [str(v) for v in desc],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    most, least, *refused = [int(v) for v in r.stdout.split()]
    assert most > least                    # by the tapes, which the least does without
    assert not refused
