"""Which kernels a float call launches, on the CPU: the built library with stand-ins for the HIP calls of its launchers, which write
down the names of the kernels and their grids."""
import ctypes
import os
import subprocess
import sys

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build

STANDIN = r"""
#include <stddef.h>
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim;
static struct { const void *host; const char *name; } known[512];
static int n_known;
static dim grid;
char launched[4096];
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, unsigned limit, void *a, void *b, void *c, void *d,
                           int *e)
{
    (void)m; (void)device; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (n_known < 512) known[n_known].host = host, known[n_known++].name = name;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int what, int d) { (void)what; (void)d; *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int what, int v) { (void)f; (void)what; (void)v; return 0; }
int __hipPushCallConfiguration(dim g, dim b, size_t m, void *s) { (void)b; (void)m; (void)s; grid = g; return 0; }
int __hipPopCallConfiguration(dim *g, dim *b, size_t *m, void **s)
{
    *g = grid;
    *b = (dim){1, 1, 1};
    *m = 0;
    *s = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dim g, dim b, void **a, size_t m, void *s)
{
    (void)b; (void)a; (void)m; (void)s;
    for (int i = 0; i < n_known; ++i)
        if (known[i].host == f) {
            const size_t at = strlen(launched);
            snprintf(launched + at, sizeof(launched) - at, "%s %u\n", known[i].name, g.x);
        }
    return 0;
}
"""

CHILD = r"""
import ctypes, re, sys
standin, lib = ctypes.CDLL(sys.argv[1]), ctypes.CDLL(sys.argv[2])
class Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "n_tree", "max_prefix_len", "dtype")] + \
        [("softmax_scale", ctypes.c_float)] + [(n, ctypes.c_int64 * 3) for n in ("q", "o", "kc", "vc", "kt", "vt")]
assert ctypes.sizeof(Desc) == int(sys.argv[3])
vp, i32 = ctypes.c_void_p, ctypes.c_int32
lib.ls_hybrid_tree_attn.argtypes = [vp] * 11 + [ctypes.c_size_t, vp]
lib.ls_prefix_attn_splitkv.argtypes = [vp] * 5 + [i32, i32, vp, vp, vp]
text = (ctypes.c_char * 4096).in_dll(standin, "launched")
at = [(i + 1) << 44 for i in range(10)]
def desc(hq, hkv, d, t, capacity):
    x = Desc(1, hq, hkv, d, t, capacity, 1, 0.0)
    for n, heads, rows in (("q", hq, t), ("o", hq, t), ("kc", hkv, capacity), ("vc", hkv, capacity), ("kt", hkv, t), ("vt", hkv, t)):
        getattr(x, n)[:] = [heads * rows * d, rows * d, d]
    return x
def kernels():
    found = []
    for line in text.value.decode().splitlines():
        name, grid = line.split()
        m = re.search(r"(float_split_kernel|merge_float_kernel)I((?:Li\d+E)+)E", name)
        found.append((m[1], *map(int, re.findall(r"Li(\d+)E", m[2])), int(grid)) if m else name)
    text.value = b""
    return found
def whole(*sizes, out=None):
    a = list(at)
    if out is not None: a[7] = out
    assert lib.ls_hybrid_tree_attn(ctypes.byref(desc(*sizes)), *a, 1 << 40, None) == 0
    return kernels()
# 64 query rows per KV head: four workgroups of 16 rows for each run of keys; head_dim, row tiles, workgroups
assert whole(4, 1, 64, 16, 100) == [("float_split_kernel", 64, 1, 4)], "one run"
assert whole(4, 1, 64, 16, 100, out=at[0]) == [("float_split_kernel", 64, 1, 4), ("merge_float_kernel", 64, 16)], "in place"
assert whole(4, 1, 64, 16, 1024) == [("float_split_kernel", 64, 1, 64), ("merge_float_kernel", 64, 16)], "16 runs"
assert whole(4, 1, 128, 16, 100)[0][:3] == ("float_split_kernel", 128, 1)
for t, n, rows in ((16, 3, 2), (4, 3, 1)):  # the stand-alone call: 32 rows per workgroup above 16 rows, no merge
    d = desc(4, 1, 64, t, 1024)
    assert lib.ls_prefix_attn_splitkv(ctypes.byref(d), *at[:4], n, 1, at[4], at[5], None) == 0
    assert kernels() == [("float_split_kernel", 64, rows, n * (4 * t // (16 * rows)))], (t, n)
print("as expected")
"""


def test_float_calls_launch_the_float_kernels(tmp_path):
    """The recording launchers of the other route tests stand in front of the choice between the float and the 16-bit kernels."""
    ls_build.build_library(force=False)
    (tmp_path / "standin.c").write_text(STANDIN)
    standin = str(tmp_path / "standin.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-Wall", "-o", standin, str(tmp_path / "standin.c")], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, standin, ls.LIB_PATH, str(ctypes.sizeof(ls.ls_desc))],
                       env=dict(os.environ, LD_PRELOAD=standin), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "as expected" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
