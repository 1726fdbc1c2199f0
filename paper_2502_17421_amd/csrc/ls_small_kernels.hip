// The small kernels of the path: tree-mask builder, masked tree attention, log-sum-exp
// merge, and the fused tree attention + merge that closes the whole call.  (LongSpec, Section 3.3; the aggregation appendix.)
#include "ls_internal.hpp"
#include "ls_tail.hpp"

namespace ls {

// --------------------------------------------------------------------------- (a) ----
// Tree mask: one workgroup per sequence; a thread walks the parent chain of its node and sets
// one bit per node met, itself included.  err_flag[b] is written 0 or 1 on every launch.
__global__ void __launch_bounds__(256)
tree_mask_kernel(const int32_t *__restrict__ parents, int32_t n_tree, uint64_t *__restrict__ mask,
                 int32_t *__restrict__ err_flag)
{
    const int b = blockIdx.x;
    const int words = (n_tree + 63) >> 6;
    build_tree_mask_rows(parents + (size_t)b * n_tree, n_tree, mask + (size_t)b * n_tree * words,
                         err_flag ? err_flag + b : nullptr, threadIdx.x, blockDim.x);
}

hipError_t launch_tree_mask(const int32_t *parents, int32_t batch, int32_t n_tree, uint64_t *mask,
                            int32_t *err_flag, hipStream_t stream)
{
    const int threads = n_tree <= 64 ? 64 : (n_tree <= 128 ? 128 : 256);
    hipLaunchKernelGGL(tree_mask_kernel, dim3(batch), dim3(threads), 0, stream, parents, n_tree, mask, err_flag);
    return hipGetLastError();
}

// Zeroes n 32-bit words (the arrival counters of the single-launch call; a kernel rather than a
// memset so that the call may sit in a captured graph).
__global__ void __launch_bounds__(256) clear_words_kernel(uint32_t *__restrict__ words, int32_t n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) words[i] = 0u;
}

hipError_t launch_clear_words(uint32_t *words, int32_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(clear_words_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, words, n);
    return hipGetLastError();
}

// --------------------------------------------------------------------------- (c) ----
// Masked tree attention: one wavefront per query row (b, h, i).  The head dimension is
// spread over the 64 lanes; the visible keys are the set bits of the row's mask, walked
// in increasing order.  Each logit is a wavefront-wide sum of per-lane products; the
// softmax state (running max, running sum) is wave-uniform.
template <typename T, int D>
__global__ void __launch_bounds__(256)
tree_attn_kernel(Problem p, const uint64_t *__restrict__ mask, Partials out)
{
    constexpr int EPL = D / kWave;  // elements per lane
    const int lane = threadIdx.x & (kWave - 1);
    const int row = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
    const int rows_total = p.batch * p.n_q_heads * p.n_tree;
    if (row >= rows_total) return;
    const int i = row % p.n_tree;
    const int h = (row / p.n_tree) % p.n_q_heads;
    const int b = row / (p.n_tree * p.n_q_heads);
    const int g = h / p.group;
    const int words = (p.n_tree + 63) >> 6;

    const T *qrow = (const T *)p.q + b * p.q_stride[0] + h * p.q_stride[1] + i * p.q_stride[2];
    const T *kbase = (const T *)p.k_tree + b * p.kt_stride[0] + g * p.kt_stride[1];
    const T *vbase = (const T *)p.v_tree + b * p.vt_stride[0] + g * p.vt_stride[1];
    const uint64_t *mrow = mask + ((size_t)b * p.n_tree + i) * words;

    float qv[EPL], acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        qv[e] = Elem<T>::load(qrow + lane * EPL + e) * p.scale_log2;
        acc[e] = 0.f;
    }
    float m_run = -INFINITY, l_run = 0.f;
    for (int w = 0; w < words; ++w) {
        uint64_t bits = mrow[w];
        if (w == words - 1 && (p.n_tree & 63)) bits &= ((uint64_t)1 << (p.n_tree & 63)) - 1;
        while (bits) {
            const int j = (w << 6) + __builtin_ctzll(bits);
            bits &= bits - 1;
            const T *krow = kbase + j * p.kt_stride[2];
            const T *vrow = vbase + j * p.vt_stride[2];
            float part = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) part += qv[e] * Elem<T>::load(krow + lane * EPL + e);
            const float z = wave_sum(part);  // base-2 logit, identical in every lane
            const float m_new = fmaxf(m_run, z);
            const float alpha = exp2f(m_run - m_new);  // 0 on the first key
            const float pj = exp2f(z - m_new);
            l_run = l_run * alpha + pj;
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                acc[e] = acc[e] * alpha + pj * Elem<T>::load(vrow + lane * EPL + e);
            m_run = m_new;
        }
    }
    const size_t prow = out.row((size_t)b * p.n_q_heads + h, 0, p.n_tree, i);
    float *orow = (float *)out.o + prow * D;
    const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) orow[lane * EPL + e] = acc[e] * inv;
    if (lane == 0) out.lse[prow] = l_run > 0.f ? (m_run + log2f(l_run)) * kLn2 : -INFINITY;
}

hipError_t launch_tree_attn(const Problem &p, int dtype, const uint64_t *mask, const Partials &out,
                            hipStream_t stream)
{
    const int rows = p.batch * p.n_q_heads * p.n_tree;
    const dim3 block(256), grid((rows + 3) / 4);
#define LS_TREE_CASE(T, DD) \
    hipLaunchKernelGGL((tree_attn_kernel<T, DD>), grid, block, 0, stream, p, mask, out)
    if (dtype == LS_BF16 && p.head_dim == 128) LS_TREE_CASE(uint16_t, 128);
    else if (dtype == LS_BF16 && p.head_dim == 64) LS_TREE_CASE(uint16_t, 64);
    else if (dtype == LS_F16 && p.head_dim == 128) LS_TREE_CASE(half_t, 128);
    else if (dtype == LS_F16 && p.head_dim == 64) LS_TREE_CASE(half_t, 64);
    else if (dtype == LS_F32 && p.head_dim == 128) LS_TREE_CASE(float, 128);
    else if (dtype == LS_F32 && p.head_dim == 64) LS_TREE_CASE(float, 64);
    else return hipErrorInvalidValue;
#undef LS_TREE_CASE
    return hipGetLastError();
}

// --------------------------------------------------------------------------- (d) ----
// Merge: one thread per (query row, 4 consecutive head-dim elements).  First pass finds
// the largest part LSE, second pass accumulates exp(LSE_k - max) weighted outputs and the
// weight sum; the result is out = sum_k w_k O_k / sum_k w_k, lse = max + log(sum_k w_k),
// which is the two-term aggregation rule of Section 3.3 applied to all parts at once.
__device__ __forceinline__ float4 load4(const float *p) { return *(const float4 *)p; }
__device__ __forceinline__ float4 load4(const uint16_t *p)
{
    const uint2 v = *(const uint2 *)p;
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xffff0000u));
}

__device__ __forceinline__ float4 load4(const half_t *p)
{
    const uint2 v = *(const uint2 *)p;
    return make_float4(half_to_float((uint16_t)v.x), half_to_float((uint16_t)(v.x >> 16)),
                       half_to_float((uint16_t)v.y), half_to_float((uint16_t)(v.y >> 16)));
}

template <typename T, typename PT, int D>
__global__ void __launch_bounds__(256)
merge_kernel(int32_t rows_total, int32_t n_q_heads, int32_t n_tree, int32_t n_parts,
             const PT *__restrict__ o_parts, const float *__restrict__ lse_parts, T *__restrict__ out,
             int64_t os0, int64_t os1, int64_t os2, float *__restrict__ lse)
{
    constexpr int TPR = D / 4;  // threads per row
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = tid / TPR;
    const int c = (tid % TPR) * 4;
    if (row >= rows_total) return;
    const int i = row % n_tree;
    const int h = (row / n_tree) % n_q_heads;
    const int b = row / (n_tree * n_q_heads);
    const size_t bh = (size_t)b * n_q_heads + h;
    const float *lp = lse_parts + bh * n_parts * n_tree + i;

    float top = -INFINITY;
    for (int k = 0; k < n_parts; ++k) top = fmaxf(top, lp[(size_t)k * n_tree]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float wsum = 0.f;
    if (top > -INFINITY) {
        for (int k = 0; k < n_parts; ++k) {
            const float l = lp[(size_t)k * n_tree];
            if (l == -INFINITY) continue;
            const float w = exp2f((l - top) * kLog2e);
            const float4 o = load4(o_parts + ((bh * n_parts + k) * n_tree + i) * D + c);
            acc.x += w * o.x;
            acc.y += w * o.y;
            acc.z += w * o.z;
            acc.w += w * o.w;
            wsum += w;
        }
    }
    const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
    T *orow = out + b * os0 + h * os1 + i * os2 + c;
    Elem<T>::store(orow + 0, acc.x * inv);
    Elem<T>::store(orow + 1, acc.y * inv);
    Elem<T>::store(orow + 2, acc.z * inv);
    Elem<T>::store(orow + 3, acc.w * inv);
    if (c == 0) lse[row] = wsum > 0.f ? top + log2f(wsum) * kLn2 : -INFINITY;
}

hipError_t launch_merge(int32_t batch, int32_t n_q_heads, int32_t n_tree, int32_t head_dim, int dtype,
                        int32_t n_parts, const void *o_parts, int parts_are_16bit, const float *lse_parts, void *out,
                        const int64_t o_stride[3], float *lse, hipStream_t stream)
{
    const int rows = batch * n_q_heads * n_tree;
    const int threads = rows * (head_dim / 4);
    const dim3 block(256), grid((threads + 255) / 256);
#define LS_MERGE_CASE(T, PT, DD)                                                                              \
    hipLaunchKernelGGL((merge_kernel<T, PT, DD>), grid, block, 0, stream, rows, n_q_heads, n_tree, n_parts,     \
                       (const PT *)o_parts, lse_parts, (T *)out, o_stride[0], o_stride[1], o_stride[2], lse)
    if (head_dim != 64 && head_dim != 128) return hipErrorInvalidValue;
    // parts are float, or 16-bit parts of a 16-bit problem in the problem's own type
    if (dtype == LS_F32) {
        if (parts_are_16bit) return hipErrorInvalidValue;
        if (head_dim == 128) LS_MERGE_CASE(float, float, 128);
        else LS_MERGE_CASE(float, float, 64);
    } else if (dtype == LS_BF16) {
        if (parts_are_16bit) {
            if (head_dim == 128) LS_MERGE_CASE(uint16_t, uint16_t, 128);
            else LS_MERGE_CASE(uint16_t, uint16_t, 64);
        } else {
            if (head_dim == 128) LS_MERGE_CASE(uint16_t, float, 128);
            else LS_MERGE_CASE(uint16_t, float, 64);
        }
    } else if (dtype == LS_F16) {
        if (parts_are_16bit) {
            if (head_dim == 128) LS_MERGE_CASE(half_t, half_t, 128);
            else LS_MERGE_CASE(half_t, half_t, 64);
        } else {
            if (head_dim == 128) LS_MERGE_CASE(half_t, float, 128);
            else LS_MERGE_CASE(half_t, float, 64);
        }
    } else {
        return hipErrorInvalidValue;
    }
#undef LS_MERGE_CASE
    return hipGetLastError();
}

// --------------------------------------------------------------------- (c) + (d) fused ----
// The kernel that ends the two-launch call: tail_rows (ls_tail.hpp) over all query rows.
// The whole-wavefront-per-row form is taken for more than 16 split rows per query row and at most
// this many rows (eight wavefronts per SIMD).
constexpr int kTailWideMaxRows = 8192;

// Waves per SIMD the compiler must leave room for (every load carries a 64-bit address of its
// own, so the register count is well above that of the data in flight).  The form for many rows
// (16 lanes per row, four 16-bit split rows per request) fits three; calls with tens of thousands of
// rows run in rounds of resident wavefronts, and a third wavefront per SIMD shortens them more
// than the registers it gives up would.
template <int LPR, int CH, int PART_BYTES> constexpr int tail_waves_per_simd()
{
    return (LPR == 16 && CH == 16) || CH * PART_BYTES >= 256 ? 1 : (LPR == 16 && CH * PART_BYTES < 128 ? 3 : 2);
}

template <typename T, int D, int LPR, int CH>
__global__ void __launch_bounds__(kWave, (tail_waves_per_simd<LPR, CH, (int)sizeof(T) * D / LPR>()))
tree_merge_kernel(Problem p, const uint64_t *__restrict__ mask, Partials parts, int32_t n_cache, T *__restrict__ out,
                  int64_t os0, int64_t os1, int64_t os2, float *__restrict__ lse)
{
    // Rows are numbered (sequence, KV head, tree node, query head within the group), so that the
    // rows of one wavefront mostly share their tree node and KV head.
    constexpr int RPW = kWave / LPR;  // query rows per wavefront
    const int lane = threadIdx.x;
    const int rows_total = p.batch * p.n_q_heads * p.n_tree;
    int r = blockIdx.x * RPW + lane / LPR;
    const bool live = r < rows_total;
    r = live ? r : rows_total - 1;  // lanes past the last row repeat it and store nothing
    const int hh = r % p.group;
    int t = r / p.group;
    const int i = t % p.n_tree;
    t /= p.n_tree;
    const int g = t % p.n_kv_heads;
    const int b = t / p.n_kv_heads;
    const uint64_t *mask_b = mask ? mask + (size_t)b * p.n_tree * ((p.n_tree + 63) >> 6) : nullptr;
    tail_rows<T, T, D, LPR, CH>(p, mask_b, parts, n_cache, out, os0, os1, os2, lse, b, g * p.group + hh, i, live, lane);
}

hipError_t launch_tree_merge(const Problem &p, int dtype, const uint64_t *mask, const Partials &cache_parts,
                             int32_t n_cache_parts, void *out, const int64_t o_stride[3], float *lse,
                             hipStream_t stream)
{
    const int rows = p.batch * p.n_q_heads * p.n_tree;
    // a whole wavefront per row: few rows, each with many split rows (see the kernel's comment)
    const bool wide = n_cache_parts > 16 && rows <= kTailWideMaxRows;
    const int rows_per_wave = wide ? 1 : 4;
    const dim3 block(kWave), grid((rows + rows_per_wave - 1) / rows_per_wave);
#define LS_TM_LAUNCH(T, DD, LPR, CH)                                                                              \
    hipLaunchKernelGGL((tree_merge_kernel<T, DD, LPR, CH>), grid, block, 0, stream, p, mask, cache_parts,         \
                       n_cache_parts, (T *)out, o_stride[0], o_stride[1], o_stride[2], lse)
#define LS_TM_CASE(T, DD)                                        \
    do {                                                         \
        if (wide) LS_TM_LAUNCH(T, DD, 64, 32);                   \
        else if (n_cache_parts <= 8) LS_TM_LAUNCH(T, DD, 16, 4); \
        else LS_TM_LAUNCH(T, DD, 16, 16);                        \
    } while (0)
    if (!cache_parts.o_is_16bit || (p.head_dim != 64 && p.head_dim != 128)) return hipErrorInvalidValue;
    if (rows <= 0) return hipSuccess;
    if (dtype == LS_BF16) {
        if (p.head_dim == 128) LS_TM_CASE(uint16_t, 128);
        else LS_TM_CASE(uint16_t, 64);
    } else if (dtype == LS_F16) {
        if (p.head_dim == 128) LS_TM_CASE(half_t, 128);
        else LS_TM_CASE(half_t, 64);
    } else {
        return hipErrorInvalidValue;  // float calls end with merge_float_kernel
    }
#undef LS_TM_CASE
#undef LS_TM_LAUNCH
    return hipGetLastError();
}

// --------------------------------------------------------------------- (d), whole path ----
// Merge of the split rows of a whole-path call whose kernels took the tree keys along (WholeCall): per
// query row n 16-bit rows side by side and their LSEs; when the call has a tree, the last one is in fp32, its
// upper halves in its place and its lower halves in the row of `out` that the merged row replaces.
//
// LG = D / 8 lanes hold a row in 16-byte pieces.  WIDE: a wavefront per query row, 64 / LG parts per
// load instruction; else LG lanes per query row (at most 8 parts).  Every load of a row is issued before
// the first is used; LSEs and rows come together, so a row costs one round trip.
//
// Bound by latency: the launch, the arguments, that round trip, and then the instructions of a wave that has its SIMD to itself
// (some 4 ns each where one waits for the other).  So the row of the tree is a step of its own, and with a wavefront
// per row a lane loads the LSEs of the parts whose rows it adds up, instead of getting weights from other lanes (69 nodes x 12k
// keys f16, 16 parts: call 35.4 -> 33.6 us; 64 rows x 32k keys, 32 parts: 35.9 -> 35.3).  With LG lanes per row the loads cost
// more than they save (eight sequences, paged: 47.4 -> 47.8).
struct MergeArgs {
    const void *o_parts;
    const float *lse_parts;
    void *out;
    float *lse;
    const SequenceSplits *table;
    int64_t o_stride[3];
    FastDiv by_tree, by_q_heads;
    int32_t n_splits, n_tree, n_q_heads, rows_total, has_tree;
};

template <int LG> __device__ __forceinline__ int max_over_groups(int x)
{
#pragma unroll
    for (int off = 32; off >= LG; off >>= 1) {
        const int y = __shfl_xor(x, off, kWave);
        x = x > y ? x : y;
    }
    return __builtin_amdgcn_readfirstlane(x);
}

// sum / max over the groups of LG lanes of a wavefront
template <int LG> __device__ __forceinline__ float groups_sum(float x)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    if constexpr (LG == 8) x += dpp_row<kRowRor8>(x);
    return x;
}
template <int LG> __device__ __forceinline__ float groups_max(float x)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    if constexpr (LG == 8) x = fmaxf(x, dpp_row<kRowRor8>(x));
    return x;
}

template <typename T, int D, bool WIDE>
__global__ void __launch_bounds__(256) merge_parts_kernel(MergeArgs a)
{
    constexpr int LG = D / 8;
    constexpr int GROUPS = kWave / LG;                    // parts (WIDE) or query rows per load instruction
    constexpr int NL = WIDE ? 64 / GROUPS : 8;            // load instructions per pass of at most 64 (8) parts
    constexpr int PASS = WIDE ? 64 : 8;
    typedef Lanes<T, 8> L8;
    // all arguments by one batch of scalar loads
    asm volatile("" ::"s"(a.o_parts), "s"(a.lse_parts), "s"(a.out), "s"(a.lse), "s"(a.table), "s"(a.o_stride[0]), "s"(a.o_stride[1]),
                 "s"(a.o_stride[2]), "s"(a.by_tree.mul), "s"(a.by_q_heads.mul), "s"(a.n_splits), "s"(a.n_tree), "s"(a.n_q_heads));
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    const int group = lane / LG, sl = lane % LG;
    int r = WIDE ? __builtin_amdgcn_readfirstlane(wave) : wave * GROUPS + group;
    if (WIDE && r >= a.rows_total) return;
    const bool live = r < a.rows_total;
    r = live ? r : a.rows_total - 1;
    const int bh = (int)a.by_tree.div((uint32_t)r), i = r - bh * a.n_tree;
    const int b = (int)a.by_q_heads.div((uint32_t)bh), h = bh - b * a.n_q_heads;
    T *orow = (T *)a.out + b * a.o_stride[0] + h * a.o_stride[1] + i * a.o_stride[2] + sl * 8;
    int n_splits = a.n_splits;                            // of this lane's row
    size_t part0 = (size_t)r * n_splits;
    if (a.table) {
        const SequenceSplits mine = a.table[b];
        const int per_seq = a.n_q_heads * a.n_tree;
        n_splits = mine.count;
        part0 = (size_t)mine.first * per_seq + (size_t)(r - b * per_seq) * n_splits;
    }
    const T *rows = (const T *)a.o_parts + part0 * D + sl * 8;
    const float *lses = a.lse_parts + part0;

    // the part with the tree keys, in fp32: the last one
    const int n_cached = n_splits - (a.has_tree ? 1 : 0);
    const int n_top = WIDE ? n_cached : max_over_groups<LG>(n_cached);  // wave-uniform
    float l_tree = -INFINITY;
    RawVec<16> high{}, low{};
    if (a.has_tree) {
        l_tree = lses[n_cached];
        high = load_raw<16>(rows + (size_t)n_cached * D);
        low = load_raw<16>(orow);
    }
    float o[8], top = l_tree, wsum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
    // a part without weight may hold anything
    auto add = [&](float weight, const float (&v)[8]) __attribute__((always_inline)) {
        wsum += weight;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = __builtin_fmaf(weight, v[e], o[e]);
    };
    auto weight_of = [&](float l) __attribute__((always_inline)) {
        return l == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((l - top) * kLog2e);
    };
    for (int k0 = 0; k0 < n_top; k0 += PASS) {
        constexpr int NLSE = WIDE ? NL : 1;               // WIDE: the LSEs of this lane's parts; else that of part sl of its row
        float l[NLSE];
        RawVec<16> raw[NL];
#pragma unroll
        for (int k = 0; k < NLSE; ++k) {
            const int part = k0 + (WIDE ? k * GROUPS + group : sl);
            l[k] = (WIDE || sl < PASS) && part < n_cached ? lses[part] : -INFINITY;
        }
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int part = k0 + (WIDE ? k * GROUPS + group : k);
            if (k0 + (WIDE ? k * GROUPS : k) < n_top)     // wave-uniform; past the last part: a valid row, weight 0
                raw[k] = load_raw<16>(rows + (size_t)(part < n_cached ? part : n_splits - 1) * D);
        }
        float t = l[0];
#pragma unroll
        for (int k = 1; k < NLSE; ++k) t = fmaxf(t, l[k]);
        if constexpr (WIDE) {
            t = groups_max<LG>(t);
        } else {
#pragma unroll
            for (int off = LG / 2; off > 0; off >>= 1) t = fmaxf(t, __shfl_xor(t, off, kWave));
        }
        t = fmaxf(t, top);
        if (k0 > 0) {                                     // what has been added up so far follows the new reference
            const float scale = top == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((top - t) * kLog2e);
            wsum *= scale;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] *= scale;
        }
        top = t;
        float w[NLSE];
#pragma unroll
        for (int k = 0; k < NLSE; ++k) w[k] = weight_of(l[k]);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            if (k0 + (WIDE ? k * GROUPS : k) < n_top) {
                const float weight = WIDE ? w[k % NLSE] : __shfl(w[0], group * LG + k, kWave);
                float v[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[k].w[e] = weight == 0.f ? 0u : raw[k].w[e];
                L8::unpack(raw[k], v);
                add(weight, v);
            }
        }
    }
    if (a.has_tree) {
        const float weight = WIDE && group > 0 ? 0.f : weight_of(l_tree);
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = weight == 0.f ? 0.f : __uint_as_float(high.w[e] << 16 | (low.w[e] & 0xffffu));
            v[2 * e + 1] = weight == 0.f ? 0.f : __uint_as_float((high.w[e] & 0xffff0000u) | low.w[e] >> 16);
        }
        add(weight, v);
    }
    if constexpr (WIDE) {
        wsum = groups_sum<LG>(wsum);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = groups_sum<LG>(o[e]);
    }
    const float inv = wsum == 0.f ? 0.f : 1.f / wsum;     // a part whose LSE is NaN makes the row and its LSE NaN
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] *= inv;
    if (live && (!WIDE || group == 0)) {
        store_raw<16>(orow, L8::pack(o));
        if (sl == 0) a.lse[r] = wsum == 0.f ? -INFINITY : top + log2f(wsum) * kLn2;
    }
}

hipError_t launch_merge_parts(const Problem &p, int dtype, const WholeCall &w, hipStream_t stream)
{
    if (dtype == LS_F32) return launch_merge_float(p, w, stream);
    const int rows = p.batch * p.n_q_heads * p.n_tree;
    const bool wide = w.n_splits > 8;
    const int rows_per_block = 4 * (wide ? 1 : kWave / (p.head_dim / 8));
    const dim3 block(256), grid((rows + rows_per_block - 1) / rows_per_block);
    const MergeArgs a{w.o_parts, w.lse_parts, w.out, w.lse, w.table, {w.o_stride[0], w.o_stride[1], w.o_stride[2]},
                      w.by_tree, w.by_q_heads, w.n_splits, p.n_tree, p.n_q_heads, rows, w.parents != nullptr};
#define LS_MP_CASE(T, DD)                                                                                   \
    do {                                                                                                    \
        if (wide) hipLaunchKernelGGL((merge_parts_kernel<T, DD, true>), grid, block, 0, stream, a);          \
        else hipLaunchKernelGGL((merge_parts_kernel<T, DD, false>), grid, block, 0, stream, a);              \
    } while (0)
    if (dtype == LS_BF16 && p.head_dim == 128) LS_MP_CASE(uint16_t, 128);
    else if (dtype == LS_BF16 && p.head_dim == 64) LS_MP_CASE(uint16_t, 64);
    else if (dtype == LS_F16 && p.head_dim == 128) LS_MP_CASE(half_t, 128);
    else if (dtype == LS_F16 && p.head_dim == 64) LS_MP_CASE(half_t, 64);
    else return hipErrorInvalidValue;
#undef LS_MP_CASE
    return hipGetLastError();
}

}  // namespace ls
