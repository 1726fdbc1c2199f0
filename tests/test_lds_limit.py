"""The kernels' dynamic LDS is allowed on each device that a process uses, and asked for again after a refusal.  On the CPU: the
built library with stand-ins for the HIP calls that its launchers make."""
import os
import subprocess
import sys

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build

STANDIN = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim;
int device, refuse, asked[8], launched[8];
int hipGetDevice(int *d) { *d = device; return 0; }
int hipDeviceGetAttribute(int *v, int what, int d) { (void)what; (void)d; *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int what, int v) { (void)f; (void)what; (void)v; ++asked[device]; return refuse; }
int __hipPushCallConfiguration(dim g, dim b, size_t m, void *s) { (void)g; (void)b; (void)m; (void)s; return 0; }
int __hipPopCallConfiguration(dim *g, dim *b, size_t *m, void **s)
{
    *g = *b = (dim){1, 1, 1};
    *m = 0;
    *s = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dim g, dim b, void **a, size_t m, void *s)
{
    (void)f; (void)g; (void)b; (void)a; (void)m; (void)s;
    ++launched[device];
    return 0;
}
"""

CHILD = r"""
import ctypes, sys
standin, lib = ctypes.CDLL(sys.argv[1]), ctypes.CDLL(sys.argv[2])
class Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "n_tree", "max_prefix_len", "dtype")] +         [("softmax_scale", ctypes.c_float)] + [(n, ctypes.c_int64 * 3) for n in ("q", "o", "kc", "vc", "kt", "vt")]
assert ctypes.sizeof(Desc) == int(sys.argv[3])
vp = ctypes.c_void_p
lib.ls_hybrid_tree_attn.argtypes = [vp] * 11 + [ctypes.c_size_t, vp]
number = lambda name, at=0: (ctypes.c_int * 8).in_dll(standin, name)[at]
for dtype, capacity in ((1, 300), (0, 300), (0, 9000)):  # the float kernel, and the two for 16-bit inputs
    d = Desc(1, 8, 2, 128, 40, capacity, dtype, 0.0)
    for n, heads, rows in (("q", 8, 40), ("o", 8, 40), ("kc", 2, capacity), ("vc", 2, capacity), ("kt", 2, 40), ("vt", 2, 40)):
        getattr(d, n)[:] = [heads * rows * 128, rows * 128, 128]
    call = lambda: lib.ls_hybrid_tree_attn(ctypes.byref(d), *[(i + 1) << 44 for i in range(10)], 1 << 40, None)
    device, refuse = ctypes.c_int.in_dll(standin, "device"), ctypes.c_int.in_dll(standin, "refuse")
    for on in (0, 1):
        device.value = on
        asked, launched = number("asked", on), number("launched", on)
        assert call() == 0 and number("asked", on) == asked + 1 and number("launched", on) > launched, (dtype, capacity, on)
        assert call() == 0 and number("asked", on) == asked + 1  # once
    device.value, refuse.value = 2, 1
    launched = number("launched", 2)
    assert call() == -7 and number("launched", 2) == launched
    refuse.value = 0
    assert call() == 0 and number("launched", 2) > launched
print("each device")
"""


def test_each_device_is_asked(tmp_path):
    if not os.path.exists(ls.LIB_PATH):
        ls_build.build_library()
    (tmp_path / "standin.c").write_text(STANDIN)
    standin = str(tmp_path / "standin.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-Wall", "-o", standin, str(tmp_path / "standin.c")], check=True)
    import ctypes
    env = dict(os.environ, LD_PRELOAD=standin)
    r = subprocess.run([sys.executable, "-c", CHILD, standin, ls.LIB_PATH, str(ctypes.sizeof(ls.ls_desc))], env=env, capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0 and "each device" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
