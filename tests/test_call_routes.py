"""Which kernels a call runs, on the CPU: the host code of the library (ls_api.hip) with launchers in place of the
kernels' that only write down what they were asked for."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2502_17421_amd import binding as ls
from paper_2502_17421_amd import build as ls_build

STUB = r"""
#include "ls_api.hip"
#include <cstdio>

static char route_text[512];
static ls::SplitPlan last_plan;
#define SAY(...) std::snprintf(route_text + std::strlen(route_text), sizeof(route_text) - std::strlen(route_text), __VA_ARGS__)

namespace ls {
hipError_t launch_wave_split(const Problem &, int, int row_tiles, const WholeCall &w, hipStream_t)
{
    SAY("wave_split(rows=%d,splits=%d%s) ", 32 * row_tiles, w.n_splits, w.parents ? ",tree" : "");
    return hipSuccess;
}
hipError_t launch_prefix_mfma(const Problem &, int, const SplitPlan &plan, const Partials &, const MaskJob &job,
                              const FusedTail &tail, hipStream_t)
{
    last_plan = plan;
    SAY("prefix(splits=%d%s%s%s%s) ", plan.n_splits, tail.parents ? ",tree" : "", job.parents ? ",mask" : "",
        plan.balanced ? ",dealt" : "", tail.counters ? ",fused" : "");
    return hipSuccess;
}
hipError_t launch_prefix_valu(const Problem &, int, const SplitPlan &plan, const Partials &, const MaskJob &, hipStream_t)
{
    SAY("float(splits=%d) ", plan.n_splits);
    return hipSuccess;
}
hipError_t launch_merge_parts(const Problem &, int, const WholeCall &, hipStream_t) { SAY("merge "); return hipSuccess; }
hipError_t launch_tree_merge(const Problem &, int, const uint64_t *mask, const Partials &, int32_t, void *, const int64_t *,
                             float *, hipStream_t)
{
    SAY(mask ? "tail " : "tail(cached) ");
    return hipSuccess;
}
hipError_t launch_tree_mask(const int32_t *, int32_t, int32_t, uint64_t *, int32_t *, hipStream_t) { SAY("mask "); return hipSuccess; }
hipError_t launch_tree_attn(const Problem &, int, const uint64_t *, const Partials &, hipStream_t) { return hipSuccess; }
hipError_t launch_merge(int32_t, int32_t, int32_t, int32_t, int, int32_t, const void *, int, const float *, void *,
                        const int64_t *, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_clear_words(uint32_t *, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_tree_accept(const int32_t *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, int32_t *,
                              int32_t *, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_commit(const Problem &, int, const int32_t *, const int32_t *, void *, void *, int32_t *, int32_t *,
                            hipStream_t) { return hipSuccess; }
int prefix_mfma_query_blocks(const Problem &p) { return (p.group * p.n_tree + 255) / 256; }
bool prefix_mfma_supports(const Problem &, int dtype) { return is_16bit(dtype); }
}  // namespace ls

extern "C" int last_row_block() { return last_plan.row_block; }
extern "C" int last_copiers() { return last_plan.copiers; }

extern "C" int count_pieces(int tiles, int piece, float reciprocal) { return ls::pieces_of(tiles, piece, reciprocal); }

extern "C" const char *take_route()
{
    static char last[512];
    std::memcpy(last, route_text, sizeof(last));
    route_text[0] = 0;
    return last;
}
"""


def build(folder, *host_flags):
    src, out = folder / "routes.hip", folder / "routes.so"
    src.write_text(STUB)
    flags = [f for f in ls_build.FLAGS if f not in ("-O3", "-Wall")]
    host = [x for f in host_flags for x in ("-Xarch_host", f)]
    subprocess.run([ls_build.HIPCC, *flags, "-O1", *host, "-o", str(out), str(src)], check=True, stderr=subprocess.DEVNULL)
    return str(out)


def load(path):
    loaded = ctypes.CDLL(path)
    loaded.take_route.restype = ctypes.c_char_p
    loaded.count_pieces.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_float]
    vp, dp = ctypes.c_void_p, ctypes.POINTER(ls.ls_desc)
    loaded.ls_hybrid_tree_attn.argtypes = [dp] + [vp] * 10 + [ctypes.c_size_t, vp]
    loaded.ls_cache_attn.argtypes = [dp] + [vp] * 7 + [ctypes.c_size_t, vp]
    loaded.ls_workspace_bytes.argtypes = [dp, ctypes.POINTER(ctypes.c_size_t)]
    return loaded


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return load(build(tmp_path_factory.mktemp("routes")))


def desc(hq, hkv, d, t, capacity, batch=1, dtype=ls.LS_BF16):
    x = ls.ls_desc()
    x.batch, x.n_q_heads, x.n_kv_heads, x.head_dim, x.n_tree, x.max_prefix_len, x.dtype = batch, hq, hkv, d, t, capacity, dtype
    for field, heads, rows in ((x.q_stride, hq, t), (x.o_stride, hq, t), (x.kc_stride, hkv, capacity), (x.vc_stride, hkv, capacity),
                               (x.kt_stride, hkv, t), (x.vt_stride, hkv, t)):
        field[0], field[1], field[2] = heads * rows * d, rows * d, d
    return x


# addresses far apart; nothing is read
Q, K, V, LENS, KT, VT, PARENTS, OUT, LSE, WORK = ((i + 1) << 44 for i in range(10))


def route(lib, x, tree=True, **at):
    a = dict(q=Q, k=K, v=V, lens=LENS, kt=KT, vt=VT, parents=PARENTS, out=OUT, lse=LSE)
    a.update(at)
    n = ctypes.c_size_t(0)
    assert lib.ls_workspace_bytes(ctypes.byref(x), ctypes.byref(n)) == 0
    if tree:
        rc = lib.ls_hybrid_tree_attn(ctypes.byref(x), a["q"], a["k"], a["v"], a["lens"], a["kt"], a["vt"], a["parents"],
                                     a["out"], a["lse"], WORK, n.value, None)
    else:
        rc = lib.ls_cache_attn(ctypes.byref(x), a["q"], a["k"], a["v"], a["lens"], a["out"], a["lse"], WORK, n.value, None)
    assert rc == 0, rc
    return lib.take_route().decode().split()


def open_ended(lib):
    for hq, hkv, t in ((4, 1, 5), (8, 1, 40)):
        x = desc(hq, hkv, 128, t, 2 ** 31 - 1)
        assert route(lib, x) == ["prefix(splits=262144,mask)", "tail"]
        assert route(lib, x, tree=False) == ["prefix(splits=262144)", "tail(cached)"]


def test_an_open_ended_capacity_does_not_overflow(tmp_path):
    """max_prefix_len is a bound and may be 2^31 - 1.  (In a child process: an overflow of the planner's integers
    traps.)"""
    path = build(tmp_path, "-fsanitize=signed-integer-overflow", "-fsanitize-trap=signed-integer-overflow")
    here = os.path.dirname(os.path.abspath(__file__))
    code = f"import sys; sys.path[:0] = [{os.path.dirname(here)!r}, {here!r}]; import test_call_routes as t; t.open_ended(t.load({path!r}))"
    done = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stderr[-2000:])


def test_a_launch_has_fewer_threads_than_hip_takes(lib):
    """One workgroup of 512 threads per sequence, head and split would be 4.9e9 threads here; the kernel that shares
    tiles has 256 per workgroup."""
    x = desc(1, 1, 64, 1, 1_200_000, batch=65535)
    assert route(lib, x) == ["prefix(splits=147,tree)", "merge"]
    assert route(lib, x, tree=False) == ["prefix(splits=147)", "merge"]


@pytest.mark.parametrize("shape", [(8, 2, 128, 8, 300), (8, 2, 128, 8, 9000), (32, 8, 128, 64, 32768)])
def test_outputs_over_inputs_take_the_route_that_reads_them_first(lib, shape):
    """What a call reads only before it writes its outputs on the tail route may lie under them: the query rows they
    replace, cached rows, lengths, parents."""
    x = desc(*shape)
    apart = route(lib, x)
    assert apart[-1] != "tail"
    cache_bytes = shape[1] * shape[4] * shape[2] * 2
    out_bytes = shape[0] * shape[3] * shape[2] * 2
    for at in ({"out": Q}, {"out": K + cache_bytes - 16}, {"out": V - out_bytes + 16}, {"out": LENS - out_bytes + 16},
               {"lse": PARENTS}, {"lse": K + 16}):
        assert route(lib, x, **at)[-1] == "tail", at
        if "lse" not in at or at["lse"] != PARENTS:
            assert route(lib, x, tree=False, **at)[-1] == "tail(cached)", at
    for at in ({"out": K + cache_bytes}, {"out": V - out_bytes}, {"out": Q + out_bytes}, {"lse": KT}):
        assert route(lib, x, **at) == apart


# query heads, KV heads, head_dim, tree nodes, capacity, sequences; whether one workgroup per 32 rows takes all keys
@pytest.mark.parametrize("shape,direct", [
    ((32, 8, 128, 48, 400, 16), True), ((32, 8, 128, 48, 400, 32), False),     # 192 rows: 768 and 1536 workgroups
    ((32, 8, 128, 400, 800, 1), True), ((32, 8, 128, 400, 800, 2), False),     # 1600 rows: 400 and 800
    ((8, 1, 128, 260, 1144, 4), False), ((8, 1, 128, 256, 1144, 4), True),     # 2080 and 2048 rows: 260 and 256
    ((32, 8, 64, 400, 800, 8), True),                                          # two of them share a compute unit
    ((32, 8, 128, 16, 400, 64), True),                                         # 64 rows: the keys are copied once
])
def test_many_row_blocks_share_their_keys(lib, shape, direct):
    assert (route(lib, desc(*shape))[0] == f"wave_split(rows={64 if shape[3] == 16 else 32},splits=1,tree)") == direct


@pytest.mark.parametrize("shape,splits", [
    ((32, 8, 128, 8, 1500, 1), 1), ((32, 8, 128, 8, 1600, 1), 13),       # 32 rows: 48 and 51 tiles
    ((32, 8, 128, 16, 730, 1), 1), ((32, 8, 128, 16, 750, 1), 6),        # 64 rows: 24 and 25
    ((32, 8, 64, 16, 990, 1), 1), ((32, 8, 64, 16, 1000, 1), 8),         # head_dim 64: 32 and 33
    ((32, 8, 128, 16, 1500, 16), 1),                                     # two splits fill the chip
])
def test_few_rows_take_one_split_where_the_merge_costs_more(lib, shape, splits):
    rows = 32 if shape[3] == 8 else 64
    assert route(lib, desc(*shape))[0] == f"wave_split(rows={rows},splits={splits},tree)"


# query heads, KV heads, head_dim, tree nodes, capacity, sequences; whether the tree keys ride on the last split
@pytest.mark.parametrize("shape,ride", [
    ((32, 8, 128, 64, 32768, 1), True), ((32, 8, 128, 64, 12000, 1), False),     # splits of less than 768 rows
    ((32, 8, 128, 256, 32768, 1), True), ((32, 8, 128, 257, 32768, 1), False),   # eight tree tiles and nine
    ((40, 8, 128, 120, 16621, 4), True), ((40, 8, 128, 120, 16621, 16), False),  # 384 workgroups and 1536
    ((40, 8, 128, 64, 16621, 32), True),                                         # two tree tiles
])
def test_trees_ride_where_that_pays(lib, shape, ride):
    got = route(lib, desc(*shape))
    assert got[0].startswith("prefix(")
    assert got[1:] == (["merge"] if ride else ["tail"]) and (",tree" in got[0]) == ride and (",mask" in got[0]) != ride
    assert (",dealt" in got[0]) == (ride and shape[5] > 1)
    assert route(lib, desc(*shape), tree=False)[1] == "merge"


def test_the_gpu_tests_reach_the_kernels_they_are_for(lib):
    import test_gpu_tree_split
    import test_gpu_wave_split
    codes = {"bf16": ls.LS_BF16, "f16": ls.LS_F16}

    def routes(cases):
        for dtype, hq, hkv, d, t, plens, *_ in cases:
            x = desc(hq, hkv, d, t, max(plens), len(plens), codes[dtype])
            yield (dtype, hq, hkv, d, t, plens), route(lib, x)

    for case, got in routes(test_gpu_wave_split.CASES):
        assert got[0].startswith("wave_split"), (case, got)
    for case, got in routes(test_gpu_tree_split.CASES):
        dealt = ",dealt" if 1 < len(case[5]) <= 32 else ""
        assert got[0].endswith(f",tree{dealt})") and got[0].startswith("prefix") and got[1:] == ["merge"], (case, got)
    for case, got in routes(test_gpu_tree_split.ON_THE_TAIL):
        assert got[0].startswith("prefix") and got[1:] == ["tail"], (case, got)


def test_pieces_are_counted_exactly_with_an_inexact_reciprocal(lib):
    """What the device deals by: ceil(tiles / piece), one at least, with a reciprocal an ulp or two off."""
    rng = np.random.default_rng(41)
    pairs = [(t, p) for p in (2, 4, 6, 10, 38, 126, 254, 256) for t in [0, 1] + [k * p + e for k in (1, 2, 3, 37, 1000) for e in (-1, 0, 1)]]
    pairs += [(int(t), int(p)) for t, p in zip(np.exp(rng.uniform(0, np.log(2 ** 24), 3000)), rng.integers(1, 5000, 3000)) if t < p * 2 ** 20]
    for tiles, piece in pairs:
        r = np.float32(1) / np.float32(piece)
        for _ in range(2):
            r = np.nextafter(r, np.float32(0))
        for _ in range(5):
            assert lib.count_pieces(tiles, piece, float(r)) == max(1, -(-tiles // piece)), (tiles, piece, r)
            r = np.nextafter(r, np.float32(1))


def test_waves_that_copy(lib):
    """At head_dim 64 a compute unit holds two blocks of 128 rows without waves that only copy, of those with them one: they go
    where no unit would have two blocks.  At head_dim 128 it holds one of either."""
    for (hq, hkv, d, t, capacity, batch), expect in (
            ((16, 16, 64, 96, 8000, 16), 1),       # 256 blocks
            ((32, 32, 64, 96, 20000, 4), 0),       # 512: four splits
            ((16, 16, 64, 128, 3000, 20), 0),      # 960: three
            ((8, 2, 64, 24, 16000, 8), 1),
            ((32, 32, 128, 96, 20000, 4), 1),      # 512
            ((8, 8, 128, 100, 20000, 40), 1)):
        route(lib, desc(hq, hkv, d, t, capacity, batch))
        assert lib.last_copiers() == expect, (hq, hkv, d, t, capacity, batch)
        assert lib.last_row_block() in (128, 256)
