"""The working copy of the parameters holds what some kernel reads: the
fragments of the streaming local-energy kernel only for models that take it
(FP32 chains from 32 units on, and 2D models whose state window does not fit
shared memory: d_h = 128, Lx > 13).  Creation over stand-ins for the device
calls, as in test_model_memory.py; the working copy is the second buffer."""
import os
import shutil
import subprocess
import sys

import pytest

from test_model_memory import LIB, STAND_INS

SCRIPT = r"""
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
shim.set_limit.argtypes = [C.c_size_t]; shim.nth.restype = C.c_size_t
class Desc(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("Lx", "Ly", "dim", "hidden", "cplx", "marshall", "zm", "dt")] + [
        ("seed", C.c_uint64), ("max_Ns", C.c_int32), ("options", C.c_int32)]
d = Desc(*[int(v) for v in sys.argv[3:]])
shim.set_limit(1 << 40)
h = C.c_void_p()
assert lib.minsr_create_model(C.byref(d), C.byref(h)) == 0
print(shim.nth(1))
"""


@pytest.mark.skipif(not os.path.exists(LIB) or not shutil.which("gcc"), reason="library or gcc missing")
@pytest.mark.parametrize("Lx,Ly,dim,H,f64,fragments", [
    (10, 10, 2, 128, False, False), (13, 2, 2, 128, False, False), (14, 2, 2, 128, False, True),
    (16, 4, 2, 64, False, False), (40, 1, 1, 32, False, True), (40, 1, 1, 16, False, False),
    (6, 6, 2, 32, True, False),
])
def test_working_copy_is_what_is_read(tmp_path, Lx, Ly, dim, H, f64, fragments):
    import paper_2608_18065_amd as pm
    (tmp_path / "s.c").write_text(STAND_INS + "size_t nth(int i) { return at[i][1]; }\n")
    so = str(tmp_path / "s.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", so, str(tmp_path / "s.c")], check=True)
    desc = (Lx, Ly, dim, H, 0, 0, 0, pm.F64 if f64 else pm.F32, 1, 16, 0)
    r = subprocess.run([sys.executable, "-c", SCRIPT, so, LIB] + [str(v) for v in desc],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    ds = 2 * dim
    n = (6 if dim == 1 else 10) * H * H + 3 * ds * H + 8 * H + 4
    if fragments:
        n += 3 * H * (H + ds) + (2 * H * H if dim == 2 else 0)
    assert int(r.stdout) == n * (8 if f64 else 4)
