// Host side of the C ABI declared in include/ls_attn.h: argument checks, split planning,
// workspace layout and kernel dispatch.  No device memory is allocated here.
#include <cmath>
#include <cstring>
#include <mutex>

#include "ls_internal.hpp"

// Workspace of ls_hybrid_tree_attn_static: one array per GPU, part of the loaded code object and
// held until the process ends.  In host code the array's name only identifies the symbol; the
// memory is reached through the per-device address that hipGetSymbolAddress returns.
static __device__ __align__(256) unsigned char scratch[LS_STATIC_SCRATCH_BYTES];

namespace ls {

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

inline size_t elem_size(int dtype) { return is_16bit(dtype) ? 2 : 4; }

int check_stride(const int64_t s[3], int head_dim, size_t esz, bool is_output)
{
    for (int a = 0; a < 3; ++a) {
        if (s[a] < 0) return LS_ERR_STRIDE;
        if ((size_t)s[a] * esz % 16 != 0) return LS_ERR_STRIDE;
    }
    if (s[2] < head_dim) return LS_ERR_STRIDE;
    if (is_output && (s[0] <= 0 || s[1] <= 0)) return LS_ERR_STRIDE;
    return LS_OK;
}

int validate(const ls_desc *d)
{
    if (!d) return LS_ERR_NULL;
    if (d->batch <= 0 || d->n_q_heads <= 0 || d->n_kv_heads <= 0 || d->head_dim <= 0 || d->n_tree <= 0 ||
        d->max_prefix_len < 0)
        return LS_ERR_SHAPE;
    if (d->n_q_heads % d->n_kv_heads != 0) return LS_ERR_SHAPE;
    if (d->dtype != LS_BF16 && d->dtype != LS_F32 && d->dtype != LS_F16) return LS_ERR_DTYPE;
    if (!(d->softmax_scale >= 0.f) || std::isinf(d->softmax_scale)) return LS_ERR_SHAPE;
    if (d->head_dim != 64 && d->head_dim != 128) return LS_ERR_UNSUPPORTED;
    if (d->n_tree > LS_MAX_TREE) return LS_ERR_UNSUPPORTED;
    if ((int64_t)d->batch * d->n_kv_heads > 65535) return LS_ERR_UNSUPPORTED;
    if ((int64_t)d->batch * d->n_q_heads * d->n_tree > (1 << 24)) return LS_ERR_UNSUPPORTED;
    const size_t esz = elem_size(d->dtype);
    int rc;
    if ((rc = check_stride(d->q_stride, d->head_dim, esz, false))) return rc;
    if ((rc = check_stride(d->o_stride, d->head_dim, esz, true))) return rc;
    if ((rc = check_stride(d->kc_stride, d->head_dim, esz, false))) return rc;
    if ((rc = check_stride(d->vc_stride, d->head_dim, esz, false))) return rc;
    if ((rc = check_stride(d->kt_stride, d->head_dim, esz, false))) return rc;
    if ((rc = check_stride(d->vt_stride, d->head_dim, esz, false))) return rc;
    return LS_OK;
}

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

Problem make_problem(const ls_desc &d, const void *q, const void *kc, const void *vc, const int32_t *plens,
                     const void *kt, const void *vt)
{
    Problem p;
    std::memset(&p, 0, sizeof(p));
    p.q = q;
    p.k_cache = kc;
    p.v_cache = vc;
    p.k_tree = kt;
    p.v_tree = vt;
    p.prefix_lens = plens;
    p.prefix_len_all = d.max_prefix_len;
    p.batch = d.batch;
    p.n_q_heads = d.n_q_heads;
    p.n_kv_heads = d.n_kv_heads;
    p.group = d.n_q_heads / d.n_kv_heads;
    p.head_dim = d.head_dim;
    p.n_tree = d.n_tree;
    p.max_prefix_len = d.max_prefix_len;
    const float scale = d.softmax_scale > 0.f ? d.softmax_scale : 1.0f / std::sqrt((float)d.head_dim);
    p.scale_log2 = scale * kLog2e;
    for (int a = 0; a < 3; ++a) {
        p.q_stride[a] = d.q_stride[a];
        p.kc_stride[a] = d.kc_stride[a];
        p.vc_stride[a] = d.vc_stride[a];
        p.kt_stride[a] = d.kt_stride[a];
        p.vt_stride[a] = d.vt_stride[a];
    }
    return p;
}

int compute_units()
{
    static int cached = 0;
    if (cached) return cached;
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
        cached = n;
    else {
        (void)hipGetLastError();
        return 256;  // MI355X; not cached so a later call with a device present asks again
    }
    return cached;
}

// The first bytes of every workspace are the arrival counters of the single-launch call, at a
// place that does not depend on the problem: one ls_workspace_init serves every later call.
constexpr size_t kArrivalBytes = (size_t)kMaxArrivalCounters * kCounterWords * sizeof(uint64_t);
static_assert(kArrivalBytes == LS_WORKSPACE_COUNTER_BYTES, "the header states the size");

// Polls a workgroup of the single-launch call spends waiting for the rest of its (sequence, KV
// head, query block) before it leaves its rows to the last one: about 20 ms.  Waiting makes sense
// only when every workgroup of the launch has a compute unit of its own from the start.
constexpr int32_t kDefaultSpinPolls = 40000;
int32_t g_spin_polls = -1;  // < 0: the default

struct Workspace {
    size_t off_mask, off_err, off_lse, off_o, total;
    int32_t n_parts;
};

Workspace layout(const ls_desc &d, const SplitPlan &plan)
{
    Workspace w;
    const size_t words = (d.n_tree + 63) / 64;
    w.n_parts = plan.n_splits;
    const size_t rows = (size_t)d.batch * d.n_q_heads * w.n_parts * d.n_tree;
    w.off_mask = align_up(kArrivalBytes);
    w.off_err = align_up(w.off_mask + (size_t)d.batch * d.n_tree * words * sizeof(uint64_t));
    w.off_lse = align_up(w.off_err + (size_t)d.batch * sizeof(int32_t));
    w.off_o = align_up(w.off_lse + rows * sizeof(float));
    w.total = align_up(w.off_o + rows * d.head_dim * elem_size(d.dtype));
    return w;
}

}  // namespace

namespace {

constexpr int kMaxDevices = 64;

// Device address of `scratch` on the current device; looked up once per device, with that
// device current.  Returns nullptr (and leaves *dev_out unset) when HIP reports an error.
void *static_scratch_of_current_device()
{
    static std::mutex lock;
    static void *ptr_of[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> guard(lock);
    if (!ptr_of[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(::scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        ptr_of[dev] = ptr;
    }
    return ptr_of[dev];
}

}  // namespace

// Split schedule.  The cached keys of every sequence are cut into pieces of split_len rows
// (a multiple of 64); the grid is sized for max_prefix_len.  Left to the library, the count S
// minimises a modelled time.  Float path: units*S workgroups run in ceil(units*S / slots)
// rounds of max_prefix_len / S keys each, plus a small charge per split; this count is that of the
// stand-alone call and of the workspace, and the most that a whole call takes (plan_float).  MFMA path: the
// time of the whole call, cached-key kernel plus the kernel that merges the S parts of every
// row, from figures measured on MI355X (microseconds; f = share of the compute units the
// launch occupies, tiles of 32 keys):
//   kernel = start-up + (rounds - 1) * 5 + rounds * tiles per workgroup * time per tile
//     query blocks of 256 rows: start-up 10.5 up to f = 1/2 and 13 at f = 1, a tile 0.60 and 0.84
//       (the matrix cores are power-limited: half the compute units get through a tile in 0.7
//       of the time that all of them take, so the second half of the chip buys 1.4x, not 2x)
//     query blocks of 128 rows: start-up 6.7 + 1.8 f, a tile 0.50 up to f = 1/2, 0.66 at f = 1
//       (the HBM rate)
//   merge  = 7 + bytes of the partial rows / 3.5 TB/s
// With it a 2048-row call over 8 KV heads takes 16 splits up to about 12k cached keys and 32
// beyond 20k (measured: 8k keys 28.9 against 32.2 us, 12k 32.9 against 39.1, 24k 47.9 against
// 45.7), because every split adds a partial row per query row to write and to merge.
SplitPlan plan_splits(const ls_desc &d, int32_t request)
{
    constexpr int kTile = 64;
    SplitPlan plan;
    const int64_t max_p = d.max_prefix_len;
    int64_t s = request;
    if (s <= 0) {
        const int group = d.n_q_heads / d.n_kv_heads;
        const int rows_kv = group * d.n_tree;
        const int rows_wg = is_16bit(d.dtype) ? kPrefixRowsPerWorkgroup : 32;
        const int64_t units = (int64_t)d.batch * d.n_kv_heads * ((rows_kv + rows_wg - 1) / rows_wg);
        const int64_t slots = (int64_t)compute_units() * (is_16bit(d.dtype) ? kPrefixWorkgroupsPerCU : 1);
        // a split is at least 64 keys (a 512-key window measured 12.8 us in two splits, 10.1 in
        // four and 8.75 in eight: the start-up of a workgroup costs more than its few tiles)
        int64_t s_max = max_p / kTile;
        if (s_max > 64) s_max = 64;
        if (s_max < 1) s_max = 1;
        double best = 0.0;
        bool have = false;
        s = 1;
        const bool mfma = is_16bit(d.dtype);
        const bool heavy = rows_kv > kPrefixRowsPerWorkgroup / 2;
        const double rows_total = (double)d.batch * d.n_q_heads * d.n_tree;
        for (int64_t cand = 1; cand <= s_max; ++cand) {
            int64_t len_c = ((max_p + cand - 1) / cand + kTile - 1) / kTile * kTile;
            if (len_c < kTile) len_c = kTile;
            int64_t n_c = (max_p + len_c - 1) / len_c;  // the count this candidate ends up with
            if (n_c < 1) n_c = 1;
            const int64_t rounds = (units * n_c + slots - 1) / slots;
            double cost;
            if (!mfma) {
                cost = (double)rounds / (double)cand + 0.0005 * (double)cand;
            } else {
                const double f = rounds > 1 ? 1.0 : (double)(units * n_c) / (double)slots;
                const double over = f > 0.5 ? f - 0.5 : 0.0;
                const double tile = heavy ? 0.60 + 0.48 * over : 0.50 + 0.32 * over;
                const double start = heavy ? 10.5 + 5.0 * over : 6.7 + 1.8 * f;
                const double kernel = start + 5.0 * (double)(rounds - 1) + (double)rounds * (double)(len_c / 32) * tile;
                const double merge = 7.0 + rows_total * (double)n_c * d.head_dim * 2.0 / 3.5e6;
                cost = kernel + merge;
            }
            if (mfma && len_c > kMaxSplitLen && cand < s_max) continue;  // longer than a split may be (below)
            // more splits only for a modelled gain that is more than noise (0.05 us; the float path's
            // cost is a ratio, of order 1/S)
            if (!have || cost < best - (mfma ? 0.05 : 1e-9)) {
                have = true;
                best = cost;
                s = cand;
            }
        }
    }
    // the MFMA kernel keeps the page ids of a split in registers, which bounds a split's length;
    // the bound is applied to contiguous caches too, so that one plan serves both layouts
    if (request <= 0 && is_16bit(d.dtype) && (max_p + s - 1) / s > kMaxSplitLen) s = (max_p + kMaxSplitLen - 1) / kMaxSplitLen;
    int64_t len = (max_p + s - 1) / s;
    len = (len + kTile - 1) / kTile * kTile;
    if (len < kTile) len = kTile;
    if (request <= 0) {
        s = (max_p + len - 1) / len;
        if (s < 1) s = 1;
    }
    plan.n_splits = (int32_t)s;
    plan.split_len = (int32_t)len;
    plan.per_sequence = 0;
    plan.balanced = 0;
    // Blocks of 128 rows where twice the workgroups still have a compute unit each (see ls_prefix_mfma.hip; the mask's workgroups,
    // one per sequence, come on top and wait for one).  The model above prices blocks of 256.
    const int64_t rows_kv = (int64_t)(d.n_q_heads / d.n_kv_heads) * d.n_tree;
    const int64_t light_blocks = (int64_t)d.batch * d.n_kv_heads * ((rows_kv + 127) / 128) * s;
    plan.row_block = light_blocks <= compute_units() ? 128 : 256;
    // At head_dim 64 a compute unit holds two blocks of four waves, of four and four that copy one (162 registers per lane): with
    // more blocks than compute units the former are ahead (96 rows x 20k keys, 512 blocks 105.9 against 125.3 us; 128 rows x
    // 3000 keys, 960 blocks 67.6 / 88.0), up to one per unit the latter (96 rows x 8000 keys, 256 blocks 117.6 / 106.1).
    plan.copiers = d.head_dim == 128 || light_blocks <= compute_units();
    return plan;
}

// Schedule of the whole-path calls: as many pieces as the stand-alone cached-key call would cut,
// but on the MFMA path every sequence cuts its own length into that many (SplitPlan::per_sequence).
SplitPlan plan_call(const ls_desc &d)
{
    SplitPlan plan = plan_splits(d, 0);
    plan.per_sequence = is_16bit(d.dtype) ? 1 : 0;
    return plan;
}

// Which kernels a whole-path call runs.
struct WholePlan {
    int32_t row_tiles;  // > 0: the kernel whose waves split the keys, this many tiles of 32 query rows per workgroup (float calls: of 16)
    int32_t n_splits;   // its key splits; 1: its output is final
    // the kernel for the cached keys takes the tree keys along and a merge without a tree part follows, if
    // any (else: the tail kernel does the tree keys and the merge)
    bool ride;
};

// Whether out or lse share memory with what the whole call reads while it writes them (q, and the cached keys,
// lengths and parents, which the kernels of the tail route are done with before the first output is written): in-place
// calls take that route.  A pool of pages has no known end; only its first page is looked at.
bool outputs_overlap_inputs(const ls_desc &d, const Problem &p, const int32_t *parents, const void *out, const void *lse)
{
    auto extent = [&](const int64_t s[3], int64_t n0, int64_t n1, int64_t n2) -> uintptr_t {
        if (n2 <= 0) return 0;
        return (uintptr_t)(((n0 - 1) * s[0] + (n1 - 1) * s[1] + (n2 - 1) * s[2] + d.head_dim) * (int64_t)elem_size(d.dtype));
    };
    const uintptr_t out_bytes = extent(d.o_stride, d.batch, d.n_q_heads, d.n_tree);
    const uintptr_t lse_bytes = (uintptr_t)d.batch * d.n_q_heads * d.n_tree * sizeof(float);
    auto overlaps = [&](const void *in, uintptr_t bytes) {
        const uintptr_t i0 = (uintptr_t)in, o0 = (uintptr_t)out, l0 = (uintptr_t)lse;
        return in && bytes && ((i0 < o0 + out_bytes && o0 < i0 + bytes) || (i0 < l0 + lse_bytes && l0 < i0 + bytes));
    };
    const int64_t n0 = p.block_table ? 1 : d.batch, rows = p.block_table ? 1ll << p.page_shift : d.max_prefix_len;
    return overlaps(p.q, extent(d.q_stride, d.batch, d.n_q_heads, d.n_tree)) ||
           overlaps(p.k_cache, extent(d.kc_stride, n0, d.n_kv_heads, d.max_prefix_len ? rows : 0)) ||
           overlaps(p.v_cache, extent(d.vc_stride, n0, d.n_kv_heads, d.max_prefix_len ? rows : 0)) ||
           overlaps(p.prefix_lens, (uintptr_t)d.batch * sizeof(int32_t)) ||
           overlaps(parents, (uintptr_t)d.batch * d.n_tree * sizeof(int32_t));
}

// parents: nullptr for the cached keys alone
WholePlan plan_whole(const ls_desc &d, const SplitPlan &plan, const Problem &p, const int32_t *parents, const void *out,
                     const void *lse)
{
    const bool with_tree = parents != nullptr;
    WholePlan w{0, 0, false};
    const int rows_kv = d.n_q_heads / d.n_kv_heads * d.n_tree;
    const int64_t tiles = ((int64_t)d.max_prefix_len + 31) / 32 + (with_tree ? (d.n_tree + 31) / 32 : 0);
    // the ranges in which the kernels' divisions by multiplication are exact
    const int64_t heads = (int64_t)d.batch * d.n_q_heads;
    if (heads * d.n_tree * d.n_tree >= (1ll << 32) || heads * d.n_q_heads >= (1ll << 32) ||
        (tiles + plan.n_splits) * plan.n_splits >= (1ll << 32) ||
        (int64_t)d.batch * d.n_kv_heads * ((rows_kv + 31) / 32) * plan.n_splits * ((rows_kv + 31) / 32 + plan.n_splits) >= (1ll << 32))
        return w;
    // rows of the tree are addressed with 32-bit offsets inside a tile
    if (with_tree && (d.kt_stride[2] >= (1 << 24) || d.vt_stride[2] >= (1 << 24))) return w;
    if (outputs_overlap_inputs(d, p, parents, out, lse)) return w;
    // Tree keys on the last split of the cached-key kernel: a tree tile takes it about 2 us there, which nothing overlaps
    // and re-cutting the cached keys hides where splits are long; the tail kernel takes 3 to 9 us longer than the
    // merge, and does not know pieces dealt by length.  How long a split is depends on the lengths, of which the host knows
    // a bound, so the tree is kept to what a nearly empty cache bears too, and where the launch runs in many rounds
    // its tiles are hidden by nothing.  Time against the tail kernel's, 260 shapes of 65 to 512 nodes: with at most 8
    // tree tiles and four rounds 0.90 (worst 1.05) for sequences that fill 15 % of the capacity and more, 0.98 (1.16) below;
    // with 9 tiles and more 0.78 to 1.24, and up to 1.74 below 15 % (476 nodes, 1600 keys in 30k 70.7 / 123 us); beyond four
    // rounds up to 1.24 (120 nodes, 16 sequences of 13k to 17k keys 708 / 742).  One or two tiles, 32 query and 8
    // KV heads: 64 nodes, 32k keys 55.8 / 54.3 us, 300 keys in a capacity of 32k 22.1 / 20.8.
    // Below 768 rows per split the cut of the cached keys stays that of the stand-alone call: the whole call is held to
    // 2^-7 of the largest output against the path assembled from the stand-alone calls with 16-bit parts, and another
    // cut differs by two units in the last place at single elements (8k keys, 64 nodes would take 28.0 us for 30.1).
    const int tree_tiles = with_tree ? (d.n_tree + 31) / 32 : 0;
    constexpr int kRideSplitLen = 768;  // (more than the 16 tiles up to which a split takes the deep window)
    const int64_t workgroups = (int64_t)d.batch * d.n_kv_heads * ((rows_kv + 255) / 256) * plan.n_splits;
    w.ride = tree_tiles == 0 || (plan.split_len >= kRideSplitLen &&
                                 (tree_tiles <= 2 || (tree_tiles <= 8 && workgroups <= 4 * (int64_t)compute_units())));
    w.n_splits = plan.n_splits;
    // A short cache is worked through by one workgroup per row tile in less time than the merge of a split call
    // takes: with 32 rows per workgroup up to some 1500 keys (32 rows per KV head, 8 KV heads, one split against
    // the plan's: 1000 keys 11.3 / 12.0 us, 1500 14.3 / 12.3, and 15.8 on the kernel that shares tiles; 96
    // rows x 1200 keys 13.1, and 15.3 there), with 64 rows, whose waves take twice as long per tile, up to some 700 (64 rows,
    // 8 KV heads, head_dim 128: 550 keys 13.2 / 13.4, 850 14.9 / 13.8, 1500 20.0 / 14.2, and 15.4 there; head_dim 64:
    // 1000 keys 12.5 / 12.2) unless the chip is full with two splits anyway (16 sequences, 1500 keys 29.1 / 31.3).
    constexpr int kDirectTiles = 50;
    const int few_row_tiles = rows_kv <= 32 || plan.n_splits <= 2 ? kDirectTiles : (d.head_dim == 64 ? 32 : 24);
    // With more than 64 rows every 32-row workgroup copies all keys of its head again, which costs nothing while
    // the workgroups run in a round or two, the last one not nearly empty.  Measured, the 256-row kernel against this
    // one, head_dim 128: 192 rows per KV head x 1200 keys, 768 workgroups 44.3 / 43.8 us, 1536 72.0 / 95.6; 768 rows,
    // 768 workgroups 44.4 / 43.5, 1536 73.7 / 86.0; 1600 rows x 1200 keys, 400 workgroups 34.0 / 30.0, 800
    // 45.0 / 56.7; 2080 rows x 1144 keys, 260 workgroups 28.7 / 31.3.  At head_dim 64 two workgroups share a
    // compute unit and it is ahead throughout (1600 rows x 1200 keys, 3200 workgroups 102.6 / 90.4).
    const int64_t row_blocks = (int64_t)d.batch * d.n_kv_heads * ((rows_kv + 31) / 32), cus = compute_units();
    const int64_t rounds = (row_blocks + cus - 1) / cus;
    const bool few_blocks = d.head_dim == 64 || rounds == 1 ||
                            (rows_kv <= 768 ? rounds <= 3 : rounds == 2 && 4 * row_blocks >= 6 * cus);
    constexpr int kOneSplitTiles = 80, kSplitTiles = 136;
    const int few_row_splits = tiles <= few_row_tiles ? 1 : plan.n_splits;
    if (rows_kv <= 64 && (int64_t)d.batch * d.n_kv_heads * few_row_splits < (1ll << 32) / 512) {  // HIP: fewer than 2^32 threads
        // every wave of a workgroup holds all the query rows of the KV head (32 rows per KV head, 16k keys: 52.7
        // against 57.3 us; 64 rows, 32k keys: 34.6 against 35.4; 32 rows, 8k keys: 14.2 against 20.6)
        w.row_tiles = rows_kv <= 32 ? 1 : 2;
        w.n_splits = few_row_splits;
        w.ride = true;
    } else if (tiles <= kDirectTiles && few_blocks) {
        w.row_tiles = 1;
        w.n_splits = 1;
        w.ride = true;
    } else {
        // More rows: while 32-row workgroups leave compute units idle, up to some 4k keys, the start of the kernel
        // that shares tiles (first window, 256 rows) costs more than its faster tiles save.  Measured, that
        // kernel against this one: 256 rows per KV head, 8 KV heads: 2k keys 19.3 / 14.8 us, 4k 22.3 / 17.9, 8k
        // 28.5 / 26.1 (and 35 / 41 at 16k); 96 rows: 15.2 / 12.4, 17.1 / 14.0; one split of 1024 rows x 2k keys
        // 30.4 / 19.8, of 640 rows 25.3 / 17.3.  (The limit stays below 8k keys, where this kernel is still ahead, for the
        // cut of the cached keys, as above.)
        const int64_t fit = cus / row_blocks;  // splits that fit the chip at once
        if (tiles <= (fit >= 2 ? kSplitTiles : kOneSplitTiles) && fit >= 1) {
            w.row_tiles = 1;
            w.n_splits = fit < plan.n_splits ? (int32_t)fit : plan.n_splits;
            w.ride = true;
        }
    }
    return w;
}

// Float calls: one form, so only its sizes are chosen: 16 or 32 query rows per workgroup, and into how many runs of
// 16-key tiles the keys of a sequence are cut.  Modelled time (microseconds, measured on MI355X):
//   rounds of workgroups * (2 (32 rows: 3) + tiles of a workgroup / 8 * t), t = 1.4 (2.65) at head_dim 64, 3.05 (4.9) at 128;
//   the last run holds all tree tiles, so a workgroup has as many at least (2 KV heads x 512 rows x 1000 keys, head_dim 128: 3
//   runs 27.2 us, 8 runs, the choice by equal shares, 37.7)
//   more than one run: 2.9 (head_dim 64) or 3.3 for the merge and its launch, and the parts at 3.5 TB/s
// Both row counts and all run counts against this choice, 22 shapes: within 8 % of the best one (1024 keys x 64 rows, head_dim
// 64, 1, 9 and 16 runs 18.4, 10.0 and 9.6 us; 8 KV heads x 64 rows x 1024 keys, head_dim 128, 1, 5 and 8 runs 32.7,
// 16.8 and 13.9; 8 sequences x 8 KV heads x 160 rows x 4096 keys, 1, 2 and 4 runs of 32 rows 327, 267 and 246, of 16 rows 314, 286).
WholePlan plan_float(const ls_desc &d, const SplitPlan &plan, bool with_tree)
{
    const int64_t rows_kv = (int64_t)(d.n_q_heads / d.n_kv_heads) * d.n_tree, cus = compute_units();
    const int64_t tree_tiles = with_tree ? (d.n_tree + 15) / 16 : 0, tiles = (d.max_prefix_len + 15ll) / 16 + tree_tiles;
    const bool wide = d.head_dim == 128;
    const double part_us = (double)d.batch * d.n_q_heads * d.n_tree * d.head_dim * 4.0 / 3.5e6;
    WholePlan w{0, 0, true};
    double best = 0.0;
    for (int rt = 1; rt <= 2; ++rt) {
        const int64_t units = (int64_t)d.batch * d.n_kv_heads * ((rows_kv + 16 * rt - 1) / (16 * rt));
        const double start = rt == 1 ? 2.0 : 3.0, tile = (wide ? (rt == 1 ? 3.05 : 4.9) : (rt == 1 ? 1.4 : 2.65)) / 8.0;
        auto consider = [&](int64_t n) {
            n = n < 1 ? 1 : (n > plan.n_splits ? plan.n_splits : n);
            const int64_t share = (tiles + n - 1) / n;
            const double rounds = (double)((units * n + cus - 1) / cus), per = (double)(share > tree_tiles ? share : tree_tiles);
            const double cost = rounds * (start + per * tile) + (n > 1 ? (wide ? 3.3 : 2.9) + (double)n * part_us : 0.0);
            if (w.row_tiles == 0 || cost < best) {
                best = cost;
                w.row_tiles = rt;
                w.n_splits = (int32_t)n;
            }
        };
        for (int64_t per = 4; per < tiles; per += per < 16 ? 4 : per / 2) consider((tiles + per - 1) / per);
        for (int64_t rounds = 1; rounds <= 6; ++rounds) consider(rounds * cus / units);
    }
    return w;
}

}  // namespace ls

using namespace ls;

extern "C" {

int ls_version(void) { return 100; }

// Which header this was compiled with (a hash, given by the build): callers with compiled-in signatures compare it with theirs.
#ifndef LS_INTERFACE_ID
#define LS_INTERFACE_ID ""
#endif
extern const char ls_interface_id[17] = LS_INTERFACE_ID;

const char *ls_status_string(int status)
{
    switch (status) {
    case LS_OK: return "ok";
    case LS_ERR_NULL: return "a required pointer is NULL";
    case LS_ERR_SHAPE: return "a size is non-positive or inconsistent";
    case LS_ERR_DTYPE: return "unknown dtype";
    case LS_ERR_STRIDE: return "stride or pointer breaks the 16-byte row alignment";
    case LS_ERR_TREE: return "parents is not a topologically ordered forest";
    case LS_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case LS_ERR_HIP: return "HIP reported a launch error";
    case LS_ERR_UNSUPPORTED: return "request outside the supported set";
    default: return "unknown status";
    }
}

int ls_validate_desc(const ls_desc *desc) { return validate(desc); }

int ls_validate_parents_host(const int32_t *parents, int32_t batch, int32_t n_tree)
{
    if (!parents) return LS_ERR_NULL;
    if (batch <= 0 || n_tree <= 0) return LS_ERR_SHAPE;
    for (int32_t b = 0; b < batch; ++b)
        for (int32_t i = 0; i < n_tree; ++i) {
            const int32_t p = parents[(size_t)b * n_tree + i];
            if (p < -1 || p >= i) return LS_ERR_TREE;
        }
    return LS_OK;
}

int ls_prefix_num_splits(const ls_desc *desc, int32_t *n_splits_out)
{
    if (!n_splits_out) return LS_ERR_NULL;
    const int rc = validate(desc);
    if (rc) return rc;
    *n_splits_out = plan_splits(*desc, 0).n_splits;
    return LS_OK;
}

int ls_prefix_split_len(const ls_desc *desc, int32_t n_splits, int32_t *split_len_out)
{
    if (!split_len_out) return LS_ERR_NULL;
    const int rc = validate(desc);
    if (rc) return rc;
    if (n_splits < 0) return LS_ERR_SHAPE;
    *split_len_out = plan_splits(*desc, n_splits).split_len;
    return LS_OK;
}

int ls_workspace_bytes(const ls_desc *desc, size_t *bytes_out)
{
    if (!bytes_out) return LS_ERR_NULL;
    const int rc = validate(desc);
    if (rc) return rc;
    *bytes_out = layout(*desc, plan_call(*desc)).total;
    return LS_OK;
}

int ls_workspace_error(const ls_desc *desc, void *workspace, int32_t **err_out)
{
    if (!workspace || !err_out) return LS_ERR_NULL;
    const int rc = validate(desc);
    if (rc) return rc;
    *err_out = (int32_t *)((char *)workspace + layout(*desc, plan_call(*desc)).off_err);
    return LS_OK;
}

int ls_build_tree_mask(const int32_t *parents, int32_t batch, int32_t n_tree, uint64_t *mask,
                       int32_t *err_flag, void *stream)
{
    if (!parents || !mask) return LS_ERR_NULL;
    if (batch <= 0 || n_tree <= 0) return LS_ERR_SHAPE;
    if (n_tree > LS_MAX_TREE || batch > 65535) return LS_ERR_UNSUPPORTED;
    return launch_tree_mask(parents, batch, n_tree, mask, err_flag, (hipStream_t)stream) == hipSuccess
               ? LS_OK
               : LS_ERR_HIP;
}

int ls_prefix_attn_splitkv(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                           const int32_t *prefix_lens, int32_t n_splits, int32_t part_dtype, void *o_part,
                           float *lse_part, void *stream)
{
    const int rc = validate(desc);
    if (rc) return rc;
    if (!q || !prefix_lens || !o_part || !lse_part) return LS_ERR_NULL;
    if (desc->max_prefix_len > 0 && (!k_cache || !v_cache)) return LS_ERR_NULL;
    if (n_splits < 0 || n_splits > 65535) return LS_ERR_SHAPE;
    if (part_dtype != LS_F32 && !(is_16bit(part_dtype) && part_dtype == desc->dtype)) return LS_ERR_DTYPE;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(o_part)) return LS_ERR_STRIDE;
    const SplitPlan plan = plan_splits(*desc, n_splits);
    const Problem p = make_problem(*desc, q, k_cache, v_cache, prefix_lens, nullptr, nullptr);
    const Partials out{o_part, lse_part, plan.n_splits, 0, is_16bit(part_dtype)};
    hipError_t e;
    if (prefix_mfma_supports(p, desc->dtype)) {
        e = launch_prefix_mfma(p, desc->dtype, plan, out, MaskJob{nullptr, nullptr, nullptr}, FusedTail{}, (hipStream_t)stream);
    } else {
        if (part_dtype != LS_F32) return LS_ERR_UNSUPPORTED;
        e = launch_prefix_valu(p, desc->dtype, plan, out, MaskJob{nullptr, nullptr, nullptr}, (hipStream_t)stream);
    }
    return e == hipSuccess ? LS_OK : LS_ERR_HIP;
}

int ls_tree_attn_masked(const ls_desc *desc, const void *q, const void *k_tree, const void *v_tree,
                        const uint64_t *mask, float *o_tree, float *lse_tree, void *stream)
{
    const int rc = validate(desc);
    if (rc) return rc;
    if (!q || !k_tree || !v_tree || !mask || !o_tree || !lse_tree) return LS_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_tree) || !aligned16(v_tree) || !aligned16(o_tree)) return LS_ERR_STRIDE;
    const Problem p = make_problem(*desc, q, nullptr, nullptr, nullptr, k_tree, v_tree);
    const Partials out{o_tree, lse_tree, 1, 0, 0};
    return launch_tree_attn(p, desc->dtype, mask, out, (hipStream_t)stream) == hipSuccess ? LS_OK : LS_ERR_HIP;
}

int ls_lse_merge(const ls_desc *desc, int32_t n_parts, int32_t part_dtype, const void *o_parts,
                 const float *lse_parts, void *out, float *lse, void *stream)
{
    const int rc = validate(desc);
    if (rc) return rc;
    if (!o_parts || !lse_parts || !out || !lse) return LS_ERR_NULL;
    if (n_parts <= 0) return LS_ERR_SHAPE;
    if (part_dtype != LS_F32 && !(is_16bit(part_dtype) && part_dtype == desc->dtype)) return LS_ERR_DTYPE;
    if (!aligned16(o_parts) || !aligned16(out)) return LS_ERR_STRIDE;
    return launch_merge(desc->batch, desc->n_q_heads, desc->n_tree, desc->head_dim, desc->dtype, n_parts, o_parts,
                        is_16bit(part_dtype), lse_parts, out, desc->o_stride, lse, (hipStream_t)stream) == hipSuccess
               ? LS_OK
               : LS_ERR_HIP;
}

}  // extern "C"

namespace {
// Whole-path call whose tree keys are taken along by the kernel for the cached keys, and the merge of the
// parts unless a single split's output is final.
int run_whole(const ls_desc &d, const Problem &p, SplitPlan splits, const WholePlan &plan, const int32_t *parents,
              int32_t *err, void *out, float *lse, void *o_parts, float *lse_parts, SequenceSplits *table, hipStream_t s)
{
    WholeCall w{parents, err, out, {d.o_stride[0], d.o_stride[1], d.o_stride[2]}, lse, o_parts, lse_parts, plan.n_splits,
                FastDiv::of(plan.n_splits), FastDiv::of(d.n_tree), FastDiv::of(d.n_kv_heads), FastDiv::of(d.n_q_heads), nullptr, plan.n_splits > 1};
    if (plan.row_tiles > 0) {
        // (a float call's outputs may lie over its inputs: the merge writes them when the inputs have been read)
        if (d.dtype == LS_F32 && !w.in_parts) w.in_parts = outputs_overlap_inputs(d, p, parents, out, lse);
        if (launch_wave_split(p, d.dtype, plan.row_tiles, w, s) != hipSuccess) return LS_ERR_HIP;
        if (!w.in_parts) return LS_OK;
    } else {
        const Partials parts{o_parts, lse_parts, plan.n_splits, 0, 1, 1};
        FusedTail tail{};
        tail.parents = parents;
        tail.out = out;
        for (int i = 0; i < 3; ++i) tail.o_stride[i] = d.o_stride[i];
        tail.err_flag = err;
        // several sequences: pieces dealt by length (a single piece each cannot be)
        if (d.batch > 1 && d.batch <= kMaxBalanced && p.prefix_lens && splits.n_splits > 1) {
            splits.balanced = 1;
            tail.table = table;
            w.table = table;
        }
        if (launch_prefix_mfma(p, d.dtype, splits, parts, MaskJob{nullptr, nullptr, nullptr}, tail, s) != hipSuccess)
            return LS_ERR_HIP;
    }
    return launch_merge_parts(p, d.dtype, w, s) == hipSuccess ? LS_OK : LS_ERR_HIP;
}

// The whole path for a contiguous cache.  prefix_lens: device array, or nullptr with every
// sequence holding prefix_len_all cached rows.
int hybrid_contiguous(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                      const int32_t *prefix_lens, int32_t prefix_len_all, const void *k_tree, const void *v_tree,
                      const int32_t *parents, void *out, float *lse, void *workspace, size_t workspace_bytes,
                      void *stream, bool single_launch = false)
{
    const int rc = validate(desc);
    if (rc) return rc;
    if (!q || !k_tree || !v_tree || !parents || !out || !lse) return LS_ERR_NULL;
    if (desc->max_prefix_len > 0 && (!k_cache || !v_cache)) return LS_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(k_tree) || !aligned16(v_tree) ||
        !aligned16(out))
        return LS_ERR_STRIDE;
    const SplitPlan plan = plan_call(*desc);
    const Workspace w = layout(*desc, plan);
    if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < w.total) return LS_ERR_WORKSPACE;

    char *base = (char *)workspace;
    uint64_t *mask = (uint64_t *)(base + w.off_mask);
    int32_t *err = (int32_t *)(base + w.off_err);
    float *lse_parts = (float *)(base + w.off_lse);
    void *o_parts = base + w.off_o;
    hipStream_t s = (hipStream_t)stream;
    Problem p = make_problem(*desc, q, k_cache, v_cache, prefix_lens, k_tree, v_tree);
    p.prefix_len_all = prefix_len_all;
    if (desc->dtype == LS_F32)
        return run_whole(*desc, p, plan, plan_float(*desc, plan, true), parents, err, out, lse, o_parts, lse_parts, nullptr, s);
    if (prefix_mfma_supports(p, desc->dtype) && !single_launch) {
        const WholePlan whole = plan_whole(*desc, plan, p, parents, out, lse);
        if (whole.ride) return run_whole(*desc, p, plan, whole, parents, err, out, lse, o_parts, lse_parts, (SequenceSplits *)mask, s);
    }

    // (b) cached keys -> parts [0, n_splits), stored in the problem's dtype; on the MFMA path
    // the same launch carries the workgroups of (a), the tree mask
    const Partials cache_out{o_parts, lse_parts, w.n_parts, 0, is_16bit(desc->dtype), 1};
    if (prefix_mfma_supports(p, desc->dtype)) {
        // Single launch: the last workgroup of each (sequence, KV head, query block) does (c) and (d)
        // for that block's rows; the mask workgroups still fill the workspace's mask and error words.
        const bool fused =
            single_launch && plan.n_splits <= 64 &&
            (int64_t)desc->batch * desc->n_kv_heads * prefix_mfma_query_blocks(p) <= kMaxArrivalCounters;
        FusedTail tail{};
        if (fused) {
            tail.counters = (uint64_t *)base;
            const int64_t n_workgroups =
                (int64_t)desc->batch * desc->n_kv_heads * prefix_mfma_query_blocks(p) * plan.n_splits;
            tail.spin_limit = n_workgroups <= compute_units() ? (g_spin_polls < 0 ? kDefaultSpinPolls : g_spin_polls) : 0;
            tail.parents = parents;
            tail.out = out;
            for (int i = 0; i < 3; ++i) tail.o_stride[i] = desc->o_stride[i];
            tail.lse = lse;
        }
        if (launch_prefix_mfma(p, desc->dtype, plan, cache_out, MaskJob{parents, mask, err}, tail, s) != hipSuccess)
            return LS_ERR_HIP;
        if (fused) return LS_OK;
    } else {
        return LS_ERR_UNSUPPORTED;  // 16-bit row strides beyond the MFMA kernel's range
    }
    // (c) tree keys and (d) merge, one wavefront per query row
    if (launch_tree_merge(p, desc->dtype, mask, cache_out, plan.n_splits, out, desc->o_stride, lse, s) != hipSuccess)
        return LS_ERR_HIP;
    return LS_OK;
}
}  // namespace

extern "C" {

int ls_hybrid_tree_attn(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                        const int32_t *prefix_lens, const void *k_tree, const void *v_tree,
                        const int32_t *parents, void *out, float *lse, void *workspace, size_t workspace_bytes,
                        void *stream)
{
    if (!prefix_lens) return LS_ERR_NULL;
    return hybrid_contiguous(desc, q, k_cache, v_cache, prefix_lens, 0, k_tree, v_tree, parents, out, lse, workspace,
                             workspace_bytes, stream);
}

int ls_hybrid_tree_attn_single(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                               int32_t prefix_len, const void *k_tree, const void *v_tree, const int32_t *parents,
                               void *out, float *lse, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!desc) return LS_ERR_NULL;
    if (desc->batch != 1 || prefix_len < 0 || prefix_len > desc->max_prefix_len) return LS_ERR_SHAPE;
    return hybrid_contiguous(desc, q, k_cache, v_cache, nullptr, prefix_len, k_tree, v_tree, parents, out, lse,
                             workspace, workspace_bytes, stream);
}

int ls_hybrid_tree_attn_static(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                               const int32_t *prefix_lens, const void *k_tree, const void *v_tree,
                               const int32_t *parents, void *out, float *lse, void *stream)
{
    if (!prefix_lens) return LS_ERR_NULL;
    const int rc = validate(desc);
    if (rc) return rc;
    // the size check comes first: a problem that does not fit is refused whatever the device says
    if (layout(*desc, plan_call(*desc)).total > (size_t)LS_STATIC_SCRATCH_BYTES) return LS_ERR_WORKSPACE;
    void *ws = static_scratch_of_current_device();
    if (!ws) return LS_ERR_HIP;
    return hybrid_contiguous(desc, q, k_cache, v_cache, prefix_lens, 0, k_tree, v_tree, parents, out, lse, ws,
                             (size_t)LS_STATIC_SCRATCH_BYTES, stream);
}

int ls_workspace_init(void *workspace, size_t workspace_bytes, void *stream)
{
    if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < kArrivalBytes) return LS_ERR_WORKSPACE;
    return launch_clear_words((uint32_t *)workspace, (int32_t)(kArrivalBytes / sizeof(uint32_t)), (hipStream_t)stream) ==
                   hipSuccess
               ? LS_OK
               : LS_ERR_HIP;
}

int ls_set_single_launch_polls(int32_t polls)
{
    if (polls > (1 << 24)) return LS_ERR_SHAPE;
    g_spin_polls = polls;
    return LS_OK;
}

int ls_hybrid_tree_attn_fused(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                              const int32_t *prefix_lens, const void *k_tree, const void *v_tree,
                              const int32_t *parents, void *out, float *lse, void *workspace, size_t workspace_bytes,
                              void *stream)
{
    if (!prefix_lens) return LS_ERR_NULL;
    return hybrid_contiguous(desc, q, k_cache, v_cache, prefix_lens, 0, k_tree, v_tree, parents, out, lse, workspace,
                             workspace_bytes, stream, true);
}

int ls_cache_attn(const ls_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                  const int32_t *prefix_lens, void *out, float *lse, void *workspace, size_t workspace_bytes,
                  void *stream)
{
    const int rc = validate(desc);
    if (rc) return rc;
    if (!q || !prefix_lens || !out || !lse) return LS_ERR_NULL;
    if (desc->max_prefix_len > 0 && (!k_cache || !v_cache)) return LS_ERR_NULL;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out)) return LS_ERR_STRIDE;
    const SplitPlan plan = plan_call(*desc);
    const Workspace w = layout(*desc, plan);
    if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < w.total) return LS_ERR_WORKSPACE;
    char *base = (char *)workspace;
    float *lse_parts = (float *)(base + w.off_lse);
    void *o_parts = base + w.off_o;
    hipStream_t s = (hipStream_t)stream;
    const Problem p = make_problem(*desc, q, k_cache, v_cache, prefix_lens, nullptr, nullptr);
    if (desc->dtype == LS_F32)
        return run_whole(*desc, p, plan, plan_float(*desc, plan, false), nullptr, nullptr, out, lse, o_parts, lse_parts, nullptr, s);
    if (!prefix_mfma_supports(p, desc->dtype)) return LS_ERR_UNSUPPORTED;
    const WholePlan whole = plan_whole(*desc, plan, p, nullptr, out, lse);
    if (whole.ride) return run_whole(*desc, p, plan, whole, nullptr, nullptr, out, lse, o_parts, lse_parts, (SequenceSplits *)(base + w.off_mask), s);
    const Partials parts{o_parts, lse_parts, w.n_parts, 0, 1, 1};
    if (launch_prefix_mfma(p, desc->dtype, plan, parts, MaskJob{nullptr, nullptr, nullptr}, FusedTail{}, s) != hipSuccess) return LS_ERR_HIP;
    // the tail kernel without a mask: merge of the split partials only
    if (launch_tree_merge(p, desc->dtype, nullptr, parts, plan.n_splits, out, desc->o_stride, lse, s) != hipSuccess)
        return LS_ERR_HIP;
    return LS_OK;
}

int ls_tree_accept_greedy(const int32_t *parents, const int32_t *draft_tokens, const int32_t *target_tokens,
                          int32_t batch, int32_t n_tree, int32_t *accept_path, int32_t *accept_len,
                          int32_t *next_token, int32_t *err_flag, void *stream)
{
    if (!parents || !draft_tokens || !target_tokens || !accept_path || !accept_len || !next_token) return LS_ERR_NULL;
    if (batch <= 0 || n_tree <= 0) return LS_ERR_SHAPE;
    if (n_tree > LS_MAX_TREE || batch > 65535) return LS_ERR_UNSUPPORTED;
    return launch_tree_accept(parents, draft_tokens, target_tokens, batch, n_tree, accept_path, accept_len, next_token,
                              err_flag, (hipStream_t)stream) == hipSuccess
               ? LS_OK
               : LS_ERR_HIP;
}

int ls_kv_commit(const ls_desc *desc, const void *k_tree, const void *v_tree, const int32_t *accept_path,
                 const int32_t *accept_len, const int32_t *prefix_lens, void *k_cache, void *v_cache,
                 int32_t *new_prefix_lens, int32_t *err_flag, void *stream)
{
    const int rc = validate(desc);
    if (rc) return rc;
    if (!k_tree || !v_tree || !accept_path || !accept_len || !prefix_lens || !k_cache || !v_cache) return LS_ERR_NULL;
    if (new_prefix_lens == prefix_lens) return LS_ERR_NULL;
    if (!aligned16(k_tree) || !aligned16(v_tree) || !aligned16(k_cache) || !aligned16(v_cache)) return LS_ERR_STRIDE;
    if ((int64_t)desc->batch * desc->n_kv_heads > 0x7fffffff) return LS_ERR_UNSUPPORTED;
    const Problem p = make_problem(*desc, nullptr, k_cache, v_cache, prefix_lens, k_tree, v_tree);
    return launch_kv_commit(p, desc->dtype, accept_path, accept_len, k_cache, v_cache, new_prefix_lens, err_flag,
                            (hipStream_t)stream) == hipSuccess
               ? LS_OK
               : LS_ERR_HIP;
}

namespace {

// page_size: a power of two >= 16; the table must cover max_prefix_len rows
int check_paging(const ls_desc *desc, const int32_t *block_table, int32_t bt_stride, int32_t page_size)
{
    if (!block_table) return LS_ERR_NULL;
    if (page_size <= 0 || bt_stride <= 0) return LS_ERR_SHAPE;
    if (page_size < 16 || (page_size & (page_size - 1)) != 0) return LS_ERR_UNSUPPORTED;
    if ((int64_t)bt_stride * page_size < desc->max_prefix_len) return LS_ERR_SHAPE;
    if (!is_16bit(desc->dtype)) return LS_ERR_UNSUPPORTED;  // the float kernel reads contiguous caches only
    return LS_OK;
}

int page_shift_of(int32_t page_size)
{
    int s = 0;
    while ((1 << s) < page_size) ++s;
    return s;
}

}  // namespace

int ls_hybrid_tree_attn_paged(const ls_desc *desc, const void *q, const void *k_pages, const void *v_pages,
                              const int32_t *block_table, int32_t bt_stride, int32_t page_size,
                              const int32_t *prefix_lens, const void *k_tree, const void *v_tree,
                              const int32_t *parents, void *out, float *lse, void *workspace, size_t workspace_bytes,
                              void *stream)
{
    int rc = validate(desc);
    if (rc) return rc;
    if (!q || !prefix_lens || !k_tree || !v_tree || !parents || !out || !lse) return LS_ERR_NULL;
    if (desc->max_prefix_len > 0 && (!k_pages || !v_pages)) return LS_ERR_NULL;
    if ((rc = check_paging(desc, block_table, bt_stride, page_size))) return rc;
    if (!aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(k_tree) || !aligned16(v_tree) ||
        !aligned16(out))
        return LS_ERR_STRIDE;
    const SplitPlan plan = plan_call(*desc);
    const Workspace w = layout(*desc, plan);
    if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < w.total) return LS_ERR_WORKSPACE;
    if (plan.split_len > kMaxSplitLen) return LS_ERR_UNSUPPORTED;
    char *base = (char *)workspace;
    uint64_t *mask = (uint64_t *)(base + w.off_mask);
    int32_t *err = (int32_t *)(base + w.off_err);
    Problem p = make_problem(*desc, q, k_pages, v_pages, prefix_lens, k_tree, v_tree);
    p.block_table = block_table;
    p.bt_stride = bt_stride;
    p.page_shift = page_shift_of(page_size);
    if (!prefix_mfma_supports(p, desc->dtype)) return LS_ERR_UNSUPPORTED;
    const Partials parts{base + w.off_o, (float *)(base + w.off_lse), w.n_parts, 0, 1, 1};
    hipStream_t s = (hipStream_t)stream;
    const WholePlan whole = plan_whole(*desc, plan, p, parents, out, lse);
    if (whole.ride) return run_whole(*desc, p, plan, whole, parents, err, out, lse, parts.o, parts.lse, (SequenceSplits *)mask, s);
    if (launch_prefix_mfma(p, desc->dtype, plan, parts, MaskJob{parents, mask, err}, FusedTail{}, s) != hipSuccess) return LS_ERR_HIP;
    if (launch_tree_merge(p, desc->dtype, mask, parts, plan.n_splits, out, desc->o_stride, lse, s) != hipSuccess)
        return LS_ERR_HIP;
    return LS_OK;
}

int ls_cache_attn_paged(const ls_desc *desc, const void *q, const void *k_pages, const void *v_pages,
                        const int32_t *block_table, int32_t bt_stride, int32_t page_size, const int32_t *prefix_lens,
                        void *out, float *lse, void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = validate(desc);
    if (rc) return rc;
    if (!q || !prefix_lens || !out || !lse) return LS_ERR_NULL;
    if (desc->max_prefix_len > 0 && (!k_pages || !v_pages)) return LS_ERR_NULL;
    if ((rc = check_paging(desc, block_table, bt_stride, page_size))) return rc;
    if (!aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(out)) return LS_ERR_STRIDE;
    const SplitPlan plan = plan_call(*desc);
    const Workspace w = layout(*desc, plan);
    if (!workspace || ((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < w.total) return LS_ERR_WORKSPACE;
    if (plan.split_len > kMaxSplitLen) return LS_ERR_UNSUPPORTED;
    char *base = (char *)workspace;
    Problem p = make_problem(*desc, q, k_pages, v_pages, prefix_lens, nullptr, nullptr);
    p.block_table = block_table;
    p.bt_stride = bt_stride;
    p.page_shift = page_shift_of(page_size);
    if (!prefix_mfma_supports(p, desc->dtype)) return LS_ERR_UNSUPPORTED;
    const Partials parts{base + w.off_o, (float *)(base + w.off_lse), w.n_parts, 0, 1, 1};
    hipStream_t s = (hipStream_t)stream;
    const WholePlan whole = plan_whole(*desc, plan, p, nullptr, out, lse);
    if (whole.ride) return run_whole(*desc, p, plan, whole, nullptr, nullptr, out, lse, parts.o, parts.lse, (SequenceSplits *)(base + w.off_mask), s);
    if (launch_prefix_mfma(p, desc->dtype, plan, parts, MaskJob{nullptr, nullptr, nullptr}, FusedTail{}, s) != hipSuccess)
        return LS_ERR_HIP;
    if (launch_tree_merge(p, desc->dtype, nullptr, parts, plan.n_splits, out, desc->o_stride, lse, s) != hipSuccess)
        return LS_ERR_HIP;
    return LS_OK;
}

int ls_kv_commit_paged(const ls_desc *desc, const void *k_tree, const void *v_tree, const int32_t *accept_path,
                       const int32_t *accept_len, const int32_t *prefix_lens, void *k_pages, void *v_pages,
                       const int32_t *block_table, int32_t bt_stride, int32_t page_size, int32_t *new_prefix_lens,
                       int32_t *err_flag, void *stream)
{
    int rc = validate(desc);
    if (rc) return rc;
    if (!k_tree || !v_tree || !accept_path || !accept_len || !prefix_lens || !k_pages || !v_pages) return LS_ERR_NULL;
    if (new_prefix_lens == prefix_lens) return LS_ERR_NULL;
    if (!block_table) return LS_ERR_NULL;
    if (page_size <= 0 || bt_stride <= 0) return LS_ERR_SHAPE;
    if ((page_size & (page_size - 1)) != 0) return LS_ERR_UNSUPPORTED;
    if ((int64_t)bt_stride * page_size < desc->max_prefix_len) return LS_ERR_SHAPE;
    if (!aligned16(k_tree) || !aligned16(v_tree) || !aligned16(k_pages) || !aligned16(v_pages)) return LS_ERR_STRIDE;
    Problem p = make_problem(*desc, nullptr, k_pages, v_pages, prefix_lens, k_tree, v_tree);
    p.block_table = block_table;
    p.bt_stride = bt_stride;
    p.page_shift = page_shift_of(page_size);
    return launch_kv_commit(p, desc->dtype, accept_path, accept_len, k_pages, v_pages, new_prefix_lens, err_flag,
                            (hipStream_t)stream) == hipSuccess
               ? LS_OK
               : LS_ERR_HIP;
}

}  // extern "C"
