// Internal declarations shared by the host API and the kernel translation units.
// Nothing here is part of the C ABI (see include/ls_attn.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "ls_attn.h"

namespace ls {

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kMaxSplitPages = 512;  // pages one key split of the MFMA kernel may touch (their ids sit in 2 KB of LDS)
constexpr int kPrefixRowsPerWorkgroup = 256;  // query rows per workgroup of the MFMA kernel (8 waves x 32 rows)
constexpr int kPrefixWorkgroupsPerCU = 1;     // workgroups resident per compute unit
constexpr int kMaxSplitLen = 8192;    // cache rows per split on the MFMA path: 512 pages of the smallest page size, 16

// Everything a kernel needs to find its operands; passed by value.
struct Problem {
    const void *q;
    const void *k_cache;
    const void *v_cache;
    const void *k_tree;
    const void *v_tree;
    const int32_t *prefix_lens;  // device, one per sequence; nullptr: every sequence has prefix_len_all rows
    int32_t prefix_len_all;
    // Paged cache (block_table != nullptr): cache row r of sequence b lives in page
    // block_table[b * bt_stride + (r >> page_shift)] at row r & (page_size - 1); kc_stride /
    // vc_stride then mean {between pages, between KV heads inside a page, between rows}.
    const int32_t *block_table;
    int32_t bt_stride, page_shift;
    int32_t batch, n_q_heads, n_kv_heads, group, head_dim, n_tree, max_prefix_len;
    float scale_log2;  // softmax scale times log2(e): logits are kept in base 2 inside kernels
    int64_t q_stride[3], kc_stride[3], vc_stride[3], kt_stride[3], vt_stride[3];
};

// Where partial results go: o [batch, n_q_heads, parts_stride, n_tree, head_dim] in float or
// in the problem's 16-bit type (o_is_16bit), lse [batch, n_q_heads, parts_stride, n_tree]
// float.  A producer writes parts [part_base, part_base + its own count).
struct Partials {
    void *o;
    float *lse;
    int32_t parts_stride;
    int32_t part_base;
    int32_t o_is_16bit;
    // 0: [.., part, tree row, ..] (the layout of the public subsystem entry points);
    // 1: [.., tree row, part, ..]: the parts of one query row lie side by side, which is what
    //    the kernel that merges them reads (the whole-path calls use this inside the workspace)
    int32_t row_major;
    // index of (b, h, part, tree row i) into lse, and times head_dim into o
    __host__ __device__ size_t row(size_t bh, int part, int n_tree, int i) const
    {
        return row_major ? (bh * n_tree + i) * parts_stride + part_base + part
                         : (bh * parts_stride + part_base + part) * n_tree + i;
    }
};

// Work appended to the launch of the kernel for 16-bit cached keys so that the whole call needs one launch less:
// extra workgroups (one per sequence) that build the tree mask.  parents == nullptr: none.
struct MaskJob {
    const int32_t *parents;
    uint64_t *mask;
    int32_t *err_flag;
};

constexpr int kMaxBalanced = 32;  // sequences of a call whose pieces are dealt by length

// Pieces of one sequence of a balanced call: the parts of its query rows, [row, piece], begin at row
// first * (rows per sequence) of the workspace's part array.
struct SequenceSplits {
    int32_t first, count;
};

// Pieces of at most `piece` tiles that `tiles` tiles take, one at least.  reciprocal: of piece, to the last bit or
// two; with it the quotient, below 2^20 here, is off by at most one.
__host__ __device__ inline int pieces_of(int tiles, int piece, float reciprocal)
{
    int n = (int)((float)tiles * reciprocal);
    n += n * piece < tiles ? 1 : 0;
    n += n * piece < tiles ? 1 : 0;
    n -= (n - 1) * piece >= tiles ? 1 : 0;
    return n > 1 ? n : 1;
}

// Single-launch form of the whole call.  The workgroups of one (sequence, KV head, query block),
// one per key split, share three 64-bit words: an arrival word (call number << 32 | workgroups
// counted in this call) and two claim words used by alternate calls (bit k: the rows of slice k
// are taken).  A workgroup counts itself in after its partial rows are written and fenced.  The
// one that completes the count zeroes the other claim word for the next call and adds
// 2^32 - n_splits to the arrival word: the count is back at zero and the call number has moved,
// which is what the others poll for, at most spin_limit times.  Whoever sees the move claims
// slice (its split index) of the block's rows with a fetch-or and does the tree attention and
// the merge for them; the workgroup that completed the count then claims every slice still free
// (workgroups that gave up, or all of them when spin_limit is 0) and does those too.  So every
// row is written exactly once, by the same code whoever writes it, and no wait is unbounded.
// counters == nullptr: the kernel only writes its partial rows; those of the last split include the
// tree keys if parents != nullptr (see WholeCall; out takes the lower halves of their values).
struct FusedTail {
    uint64_t *counters;  // three words per (sequence, KV head, query block); zero before the first call
    const int32_t *parents;
    void *out;
    int64_t o_stride[3];
    float *lse;
    int32_t spin_limit;  // polls (about half a microsecond apart) before a workgroup leaves its slice to the last one
    int32_t *err_flag;   // (tree keys of the last split) one word per sequence, or nullptr
    SequenceSplits *table;  // balanced calls: one entry per sequence, written for the merge
};
constexpr int kMaxArrivalCounters = 4096;  // (sequence, KV head, query block) triples one single-launch call may have
constexpr int kCounterWords = 3;           // 64-bit words per triple

struct SplitPlan {
    int32_t n_splits;   // parts the cached-key kernel writes
    int32_t split_len;  // cache rows per split
    // MFMA path, whole-path calls only (their parts are nobody else's business): every sequence
    // cuts ITS cached rows into n_splits equal pieces (a multiple of 32 rows, at most split_len)
    // instead of pieces of split_len rows sized for the longest sequence the cache can hold, so
    // that a short sequence keeps as many workgroups busy as a long one.
    int32_t per_sequence;
    // MFMA path, whole-path calls that end with merge_parts_kernel, several sequences: the batch * n_splits
    // pieces are dealt to the sequences by their length (see SequenceSplits), all of about the same size.
    int32_t balanced;
    int32_t row_block;  // query rows per workgroup of the matrix-core kernel, 256 or 128
    int32_t copiers;    // its blocks of 128 rows have four more waves, which copy
};

// n / d for wave-uniform or per-lane n by one multiplication, exact while n * d < 2^32 (the multiplier is
// ceil(2^32 / d), so the error n * (mul - 2^32/d) / 2^32 stays below 1/d).  d = 1 has no 32-bit
// multiplier and is a case of its own.  A 32-bit division costs some forty dependent instructions,
// and the kernels of the small calls did five before their first request (0.8 us).
struct FastDiv {
    uint32_t mul, d;
    static FastDiv of(uint32_t d) { return {d > 1 ? (uint32_t)((0x100000000ull + d - 1) / d) : 0u, d}; }
    __device__ __forceinline__ uint32_t div(uint32_t n) const { return d > 1 ? __umulhi(n, mul) : n; }
};

// Outputs of a whole-path call whose kernels take the tree keys as further key tiles.
// in_parts == 0: out and lse are final.  Else partial rows [b, head, tree row, split] in the problem's
// type with float LSEs.  The last split holds the tree keys (parents != nullptr); its rows are in fp32, of a 16-bit problem the
// upper 16 bits of each value in the partial row and the lower 16 bits in the row of `out`.
struct WholeCall {
    const int32_t *parents;  // nullptr: cached keys only
    int32_t *err_flag;       // one word per sequence, or nullptr
    void *out;
    int64_t o_stride[3];
    float *lse;
    void *o_parts;
    float *lse_parts;
    int32_t n_splits;
    FastDiv by_splits, by_tree, by_kv_heads, by_q_heads;  // divisors n_splits, n_tree, n_kv_heads, n_q_heads
    const SequenceSplits *table;  // balanced call: pieces per sequence; nullptr: n_splits each
    int32_t in_parts;             // rows leave as parts, also those of a single split
};

// Lets `kernel` have `bytes` of dynamic LDS on the current device; asked once per kernel and device (`done`: a bit per device).
// A refusal is reported and asked for again by the next call.
inline hipError_t allow_dynamic_lds(const void *kernel, int bytes, std::atomic<uint64_t> &done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
    return e;
}

// bf16 <-> float on raw 16-bit patterns (round to nearest even, NaN kept quiet).
__device__ __forceinline__ float bf16_to_float(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
__device__ __forceinline__ uint16_t float_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Element type tags: float, uint16_t (a bf16 bit pattern) and half_t (an IEEE half bit pattern).
struct half_t {
    uint16_t bits;
};
__device__ __forceinline__ float half_to_float(uint16_t v) { return (float)__builtin_bit_cast(_Float16, v); }
__device__ __forceinline__ uint16_t float_to_half(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }
inline bool is_16bit(int dtype) { return dtype == LS_BF16 || dtype == LS_F16; }

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {
    static __device__ __forceinline__ float load(const uint16_t *p) { return bf16_to_float(*p); }
    static __device__ __forceinline__ void store(uint16_t *p, float v) { *p = float_to_bf16(v); }
};

template <> struct Elem<half_t> {
    static __device__ __forceinline__ float load(const half_t *p) { return half_to_float(p->bits); }
    static __device__ __forceinline__ void store(half_t *p, float v) { p->bits = float_to_half(v); }
};

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// The tree-mask rows of one sequence, computed by the n_threads threads of a workgroup, node
// tid, tid + n_threads, ... each (all threads of the workgroup must call it; it synchronises
// them once).  A row is built one 64-bit word at a time from the highest word down: the chain
// index strictly decreases, so the walk visits the words in that order and ends after at most
// `node` steps whatever the array holds; an entry outside {-1} u [0, j) ends the walk and is
// reported.
__device__ __forceinline__ void build_tree_mask_rows(const int32_t *__restrict__ par, int32_t n_tree,
                                                     uint64_t *__restrict__ mask_rows,
                                                     int32_t *__restrict__ err_word, int tid, int n_threads)
{
    const int words = (n_tree + 63) >> 6;
    int bad = 0;
    for (int node = tid; node < n_tree; node += n_threads) {
        int j = node;
        for (int w = words - 1; w >= 0; --w) {
            uint64_t bits = 0;
            while (j >= 0 && (j >> 6) == w) {
                bits |= (uint64_t)1 << (j & 63);
                int p = par[j];
                if (p < -1 || p >= j) {
                    bad = 1;
                    p = -1;
                }
                j = p;
            }
            mask_rows[(size_t)node * words + w] = bits;
        }
    }
    const int any_bad = __syncthreads_or(bad);
    if (tid == 0 && err_word) *err_word = any_bad ? 1 : 0;
}

// Host launchers, one per kernel family.  Each returns a hipError_t from the launch.
hipError_t launch_tree_mask(const int32_t *parents, int32_t batch, int32_t n_tree, uint64_t *mask,
                            int32_t *err_flag, hipStream_t stream);
hipError_t launch_tree_attn(const Problem &p, int dtype, const uint64_t *mask, const Partials &out,
                            hipStream_t stream);
hipError_t launch_prefix_valu(const Problem &p, int dtype, const SplitPlan &plan, const Partials &out,
                              const MaskJob &mask_job, hipStream_t stream);
hipError_t launch_prefix_mfma(const Problem &p, int dtype, const SplitPlan &plan, const Partials &out,
                              const MaskJob &mask_job, const FusedTail &tail, hipStream_t stream);
// query blocks per KV head of the MFMA kernel (the arrival counters of a single-launch call are
// batch * n_kv_heads * this many)
int prefix_mfma_query_blocks(const Problem &p);
hipError_t launch_clear_words(uint32_t *words, int32_t n, hipStream_t stream);
bool prefix_mfma_supports(const Problem &p, int dtype);
SplitPlan plan_splits(const ls_desc &d, int32_t n_splits_request);
hipError_t launch_merge(int32_t batch, int32_t n_q_heads, int32_t n_tree, int32_t head_dim, int dtype,
                        int32_t n_parts, const void *o_parts, int parts_are_16bit, const float *lse_parts, void *out,
                        const int64_t o_stride[3], float *lse, hipStream_t stream);
// Masked tree attention and the merge with n_cache_parts cached-key partials in one kernel.
hipError_t launch_tree_merge(const Problem &p, int dtype, const uint64_t *mask, const Partials &cache_parts,
                             int32_t n_cache_parts, void *out, const int64_t o_stride[3], float *lse,
                             hipStream_t stream);

// Whole-path kernel whose waves split the keys (32 * row_tiles query rows per workgroup, 1 or 2).
hipError_t launch_wave_split(const Problem &p, int dtype, int row_tiles, const WholeCall &w, hipStream_t stream);
// The same in fp32 (16 * row_tiles query rows per workgroup), what launch_wave_split runs for LS_F32; the stand-alone call's pieces
// of plan.split_len rows, what launch_prefix_valu runs for it; and the merge of the whole path's parts, what launch_merge_parts runs.
hipError_t launch_float_split(const Problem &p, int row_tiles, const WholeCall &w, hipStream_t stream);
hipError_t launch_float_pieces(const Problem &p, const SplitPlan &plan, const Partials &out, hipStream_t stream);
hipError_t launch_merge_float(const Problem &p, const WholeCall &w, hipStream_t stream);
// Merge of the parts of a whole-path call (w.in_parts) into out / lse.
hipError_t launch_merge_parts(const Problem &p, int dtype, const WholeCall &w, hipStream_t stream);

hipError_t launch_tree_accept(const int32_t *parents, const int32_t *draft_tokens, const int32_t *target_tokens,
                              int32_t batch, int32_t n_tree, int32_t *accept_path, int32_t *accept_len,
                              int32_t *next_token, int32_t *err_flag, hipStream_t stream);
hipError_t launch_kv_commit(const Problem &p, int dtype, const int32_t *accept_path, const int32_t *accept_len,
                            void *k_cache, void *v_cache, int32_t *new_prefix_lens, int32_t *err_flag,
                            hipStream_t stream);


}  // namespace ls
