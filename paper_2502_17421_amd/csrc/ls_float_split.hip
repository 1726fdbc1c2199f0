// Attention over the cached keys and the tree in fp32 (step (b) with (c), and the merge of the parts): products on
// the matrix cores with fp32 operands and sums (v_mfma_f32_16x16x4_f32), so nothing is rounded to fewer bits.
//
// Work decomposition.  A workgroup owns (sequence, KV head, 16 * RT query rows, key split); its eight waves hold the same
// query rows and take the 16-key tiles of the split in turn, cached tiles first, then (last split) those of the tree.
// Nothing is staged: both products read their operands from global memory straight in the layout of the matrix
// instruction, because the order of a contraction and the numbering of the output columns are free:
//   S^T = K Q^T: lane (i, k), i = lane % 16, k = lane / 16, holds columns 16u + 4k .. + 3 of key row i and of query row i,
//     16 bytes per u; step (u, j) contracts columns 16u + 4k + j, k = 0..3.
//   S^T leaves lane (i, k) with keys 4k + e of query i, which is the operand of step e of
//   O^T = V^T P^T: lane (i, k) holds columns 64h + 4i .. + 3 of value row 4k + e, 256 bytes of a row per 16 lanes.  Output
//     tile (h, j) has columns 64h + 4 * row + j, so a lane ends with 16-byte pieces of the output row.
// The waves are merged through LDS in wave order, the splits by merge_float_kernel, by the aggregation rule.
//
// What bounds it.  A tile costs RT * D / 2 matrix instructions of 32 cycles.  Many keys: eight tiles of 32 rows take a workgroup
// 4.9 us at head_dim 128, of which the matrix cores need 3.9 (16 rows: 3.05 and 1.95; head_dim 64: 2.65 and 1.4 us); a second
// register set, with the tile after next on its way too, changed nothing.  Few keys: launch, first loads, a tile or two, merge.
// Against the kernel on the vector ALUs and the tail kernel that it replaces (microseconds per call, 56 shapes 1.25 to 4.0
// times as fast, none slower): 64 rows x 1024 keys, head_dim 64, 13.7 -> 9.4; 80 rows x 86 keys 15.6 -> 7.1; 8 KV heads x 108 rows
// x 1016 keys 45.0 -> 18.0; x 160 rows x 4096 keys, 8 sequences, 541 -> 250 (86 TFLOP/s).  Error against float64, relative 2-norm,
// below what it was on every one of them (3.5e-7 -> 3.0e-7, 3.6e-7 -> 2.6e-7, 4.3e-7 -> 3.3e-7, 3.8e-7 -> 3.4e-7): scores are four
// sums, and outputs sums in two levels.  Runs of eight tiles instead of four: the last one 3.7e-7 and 1 % less time, but 8 KV heads
// x 256 rows x 4000 keys at head_dim 64 3.7e-7, where it was 3.6e-7 (now 3.5e-7); without levels 4.9e-7.
#include "ls_internal.hpp"
#include "ls_mfma.hpp"

namespace ls {

namespace {

constexpr int FTK = 16;             // keys per tile
constexpr int FNW = 8;              // waves per workgroup
constexpr int kChain = 4;           // tiles a wave adds up before it puts the sums aside
constexpr float kFloatRaise = 8.f;  // the reference exponent is raised when a score exceeds it by 2^8
typedef float floatx4 __attribute__((ext_vector_type(4)));

// n / d for every 32-bit n: the multiplier is at most d / 2^32 too large relative to 1, so the quotient is off by one at most
__device__ __forceinline__ uint32_t divide(FastDiv by, uint32_t n)
{
    const uint32_t q = by.div(n);
    return q - (uint64_t(q) * by.d > n ? 1u : 0u);
}

// max / sum over the four lanes that hold keys of the same query
__device__ __forceinline__ float keys_max(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return half_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float keys_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return half_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

__device__ __forceinline__ bool not_finite(float x) { return !(fabsf(x) <= 3.402823466e38f); }

}  // namespace

// Strides in elements.  Row (b, head, node i) of part `split` lies at (b * n_q_heads + head) * part_h + split * part_s +
// i * part_t in lse_parts, and times head_dim in o_parts.
struct FloatArgs {
    const int32_t *prefix_lens, *parents;
    const float *q, *k_cache, *v_cache, *k_tree, *v_tree;
    int64_t q_s[3], kc_s[3], vc_s[3], kt_s[3], vt_s[3], o_s[3];
    int32_t prefix_len_all, max_prefix_len, n_tree, rows_kv, group, n_kv_heads, n_q_heads, n_splits;
    int32_t split_tiles;  // 0: every sequence cuts its own tiles into n_splits runs
    uint32_t first_item;
    FastDiv by_splits, by_tree, by_kv_heads, by_row_blocks;
    float scale_log2;
    int32_t *err_flag;
    float *out, *lse;            // final rows, if o_parts is nullptr
    float *o_parts, *lse_parts;
    int64_t part_h, part_s, part_t;
};

template <int D, int RT>
__global__ void __launch_bounds__(FNW * 64, 2)
float_split_kernel(FloatArgs a)
{
    constexpr int KU = D / 16;  // 16-byte pieces of a key row per lane
    constexpr int VH = D / 64;  // of a value row
    constexpr int PPR = D / 4;  // 16-byte pieces per row
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    float4 *o_sh = (float4 *)smem;                                        // [row tile][wave][row][piece]
    float2 *ml_sh = (float2 *)(smem + RT * FNW * 16 * D * 4);             // [row tile][row][wave]
    int32_t *par_sh = (int32_t *)(smem + RT * FNW * 16 * (D * 4 + 8));  // parents; up to 64 nodes: every node's mask
    float4 *q_sh = (float4 *)(par_sh + LS_MAX_TREE);                        // [row tile][piece][lane] (RT > 1)

    // what the first requests need, fetched by one batch of scalar loads
    asm volatile("" ::"s"(a.prefix_lens), "s"(a.q), "s"(a.k_cache), "s"(a.v_cache), "s"(a.kc_s[0]), "s"(a.kc_s[1]), "s"(a.kc_s[2]),
                 "s"(a.vc_s[0]), "s"(a.vc_s[1]), "s"(a.vc_s[2]), "s"(a.q_s[0]), "s"(a.q_s[1]), "s"(a.q_s[2]), "s"(a.parents),
                 "s"(a.max_prefix_len), "s"(a.n_tree), "s"(a.rows_kv), "s"(a.n_splits), "s"(a.split_tiles), "s"(a.by_splits.mul),
                 "s"(a.by_tree.mul), "s"(a.by_kv_heads.mul), "s"(a.by_row_blocks.mul));
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, li = lane & 15, lk = lane >> 4;

    // row blocks of the same keys on one XCD, whose L2 they share (workgroups are dealt to the eight XCDs in turn)
    uint32_t item = blockIdx.x;
    if (a.by_row_blocks.d > 1) {
        const uint32_t xcd = blockIdx.x & 7u, per_xcd = gridDim.x >> 3, extra = gridDim.x & 7u;
        item = xcd * per_xcd + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
    }
    item += a.first_item;
    const uint32_t item_split = divide(a.by_row_blocks, item);
    const uint32_t bz = divide(a.by_splits, item_split);
    const int split = (int)(item_split - bz * (uint32_t)a.n_splits);
    const int b = (int)divide(a.by_kv_heads, bz);
    const int g = (int)bz - b * a.n_kv_heads;
    const int row_block = (int)(item - item_split * a.by_row_blocks.d);
    const int row0 = row_block * (16 * RT);

    int plen = a.prefix_lens ? a.prefix_lens[b] : a.prefix_len_all;
    plen = plen < 0 ? 0 : (plen > a.max_prefix_len ? a.max_prefix_len : plen);
    const int n_splits = a.n_splits;
    const int all_pref = (plen >> 4) + ((plen & 15) ? 1 : 0);
    const int tree_tiles = a.parents ? (a.n_tree + FTK - 1) / FTK : 0;
    const bool last_split = split == n_splits - 1;
    const int per_split = a.split_tiles ? a.split_tiles : (int)divide(a.by_splits, (uint32_t)(all_pref + tree_tiles + n_splits - 1));
    const int64_t lo = (int64_t)split * per_split;
    const int t_lo = lo < all_pref ? (int)lo : all_pref;
    int t_hi = last_split && !a.split_tiles ? all_pref : (all_pref - t_lo < per_split ? all_pref : t_lo + per_split);
    const int n_pref = t_hi - t_lo;
    const int n_all = n_pref + (last_split ? tree_tiles : 0);

    const float *kc = a.k_cache + b * a.kc_s[0] + g * a.kc_s[1], *vc = a.v_cache + b * a.vc_s[0] + g * a.vc_s[1];
    const float *kt = a.k_tree + b * a.kt_s[0] + g * a.kt_s[1], *vt = a.v_tree + b * a.vt_s[0] + g * a.vt_s[1];

    // rows past the end of the cache (the tree) repeat the last one; their scores are masked
    auto first_row = [&](int t) __attribute__((always_inline)) { return (t < n_pref ? t_lo + t : t - n_pref) * FTK; };
    auto load_k = [&](int t, float4 (&k)[KU]) __attribute__((always_inline)) {
        const bool tree = t >= n_pref;
        const int last = (tree ? a.n_tree : plen) - 1, r = first_row(t) + li;
        const float *src = (tree ? kt : kc) + (int64_t)(r < last ? r : last) * (tree ? a.kt_s[2] : a.kc_s[2]) + 4 * lk;
#pragma unroll
        for (int u = 0; u < KU; ++u) k[u] = *(const float4 *)(src + 16 * u);
    };
    auto load_v = [&](int t, float4 (&v)[4][VH]) __attribute__((always_inline)) {
        const bool tree = t >= n_pref;
        const int last = (tree ? a.n_tree : plen) - 1, r0 = first_row(t) + 4 * lk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = r0 + e;
            const float *src = (tree ? vt : vc) + (int64_t)(r < last ? r : last) * (tree ? a.vt_s[2] : a.vc_s[2]) + 4 * li;
#pragma unroll
            for (int h = 0; h < VH; ++h) v[e][h] = *(const float4 *)(src + 64 * h);
        }
    };
    auto row_of = [&](int rt) __attribute__((always_inline)) {  // this lane's query row; rows past the end repeat the last
        const int m = row0 + 16 * rt + li;
        return m < a.rows_kv ? m : a.rows_kv - 1;
    };
    const bool busy = wave < n_all;
    auto q_piece = [&](int rt, int u) __attribute__((always_inline)) {  // in base-2 units
        const int m = row_of(rt), hh = (int)divide(a.by_tree, (uint32_t)m), ti = m - hh * a.n_tree;
        return (const float4 *)(a.q + b * a.q_s[0] + (g * a.group + hh) * a.q_s[1] + ti * a.q_s[2] + 4 * lk + 16 * u);
    };
    auto scaled = [&](float4 x) __attribute__((always_inline)) {
        return make_float4(x.x * a.scale_log2, x.y * a.scale_log2, x.z * a.scale_log2, x.w * a.scale_log2);
    };
    // the query operand, the same in all waves: in registers (RT == 1) or, every wave bringing its share, in LDS
    constexpr int SHARE = RT * KU / FNW;
    static_assert(RT == 1 || RT * KU % FNW == 0, "");
    float4 k[KU], v[4][VH], q[RT == 1 ? KU : SHARE];
    if (busy) load_k(wave, k);
#pragma unroll
    for (int u = 0; u < (RT == 1 ? KU : SHARE); ++u)
        q[u] = RT == 1 ? *q_piece(0, u) : *q_piece((wave * SHARE + u) / KU, (wave * SHARE + u) % KU);
    if (busy) load_v(wave, v);

    // ---- tree mask: by the waves with tree tiles, which all write the same values ------------------------
    const bool tree_wave = busy && n_all > n_pref && wave + ((n_all - 1 - wave) / FNW) * FNW >= n_pref;
    if (tree_wave) {
        bool bad_parent = false;
        const int32_t *par = a.parents + (int64_t)b * a.n_tree;
        for (int i = lane; i < (a.n_tree <= 64 ? 64 : a.n_tree); i += 64) {
            int anc = i < a.n_tree ? par[i] : -1;
            if (anc < -1 || anc >= i) {  // not a forest in topological order: treat the node as a root
                bad_parent = true;
                anc = -1;
            }
            if (a.n_tree <= 64) ((uint2 *)par_sh)[lane] = ancestor_mask(anc, lane);  // one pass, all lanes
            else par_sh[i] = anc;
        }
        if (n_pref % FNW == wave && g == 0 && row_block == 0) {  // the wave of the first tree tile reports
            const bool any_bad = __any(bad_parent);
            if (lane == 0 && a.err_flag) a.err_flag[b] = any_bad ? 1 : 0;
        }
    }

#pragma unroll
    for (int u = 0; u < (RT == 1 ? KU : SHARE); ++u) {
        q[u] = scaled(q[u]);
        if constexpr (RT > 1) q_sh[(wave * SHARE + u) * 64 + lane] = q[u];
    }
    if constexpr (RT > 1) __syncthreads();
    floatx4 o[RT][VH][4];
    float m_run[RT], l_run[RT];  // reference exponent; sum of the numerators of this lane's keys
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m_run[rt] = -INFINITY;
        l_run[rt] = 0.f;
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) o[rt][h][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // nodes of tree tile tt that query row `rt` of this lane sees, among this lane's keys
    auto visible = [&](int rt, int tt) __attribute__((always_inline)) {
        const int m = row_of(rt);
        int node = m - (int)divide(a.by_tree, (uint32_t)m) * a.n_tree;
        uint32_t word;
        if (a.n_tree <= 64) {
            word = (uint32_t)par_sh[2 * node + (tt >> 1)];
        } else {
            while (node >= (tt >> 1) * 32 + 32) node = par_sh[node];
            word = take_chain_word(par_sh, node, tt >> 1);
        }
        return word >> (16 * (tt & 1));
    };

    // Sums of more than kChain tiles are added up in two levels, the upper one in the wave's LDS rows: their rounding error
    // grows with the square root of the longest run of additions.
    float m_kept[RT];
    bool kept = false;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) m_kept[rt] = -INFINITY;
    auto o_slot = [&](int rt, int h, int e) __attribute__((always_inline)) {
        return o_sh + ((rt * FNW + wave) * 16 + li) * PPR + ((16 * h + 4 * lk + e) ^ li);
    };
    auto add_kept = [&]() __attribute__((always_inline)) {  // to the sums in registers
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const float f = m_kept[rt] == m_run[rt] ? 1.f : __builtin_amdgcn_exp2f(m_kept[rt] - m_run[rt]);
#pragma unroll
            for (int h = 0; h < VH; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 x = *o_slot(rt, h, e);
                    o[rt][h][0][e] = __builtin_fmaf(f, x.x, o[rt][h][0][e]);
                    o[rt][h][1][e] = __builtin_fmaf(f, x.y, o[rt][h][1][e]);
                    o[rt][h][2][e] = __builtin_fmaf(f, x.z, o[rt][h][2][e]);
                    o[rt][h][3][e] = __builtin_fmaf(f, x.w, o[rt][h][3][e]);
                }
        }
    };
    auto put = [&](int rt) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < VH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *o_slot(rt, h, e) = make_float4(o[rt][h][0][e], o[rt][h][1][e], o[rt][h][2][e], o[rt][h][3][e]);
    };

    int in_chain = 0;
    bool dropped = false;  // wave-uniform: infinities or NaN among the values of this wave's tree tiles
    for (int t = wave; t < n_all; t += FNW) {
        const bool tree = t >= n_pref;
        floatx4 s[RT][4];  // four chains: a score's rounding error grows with the longest
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) s[rt][0] = s[rt][1] = s[rt][2] = s[rt][3] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const float ku[4] = {k[u].x, k[u].y, k[u].z, k[u].w};
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const float4 qf = RT == 1 ? q[RT == 1 ? u : 0] : q_sh[(rt * KU + u) * 64 + lane];
                const float qu[4] = {qf.x, qf.y, qf.z, qf.w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    s[rt][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ku[j], qu[j], s[rt][j], 0, 0, 0);
            }
        }
        if (t + FNW < n_all) load_k(t + FNW, k);
        const int rest = (tree ? a.n_tree : plen) - first_row(t), valid = rest - 4 * lk;  // this lane's first `valid` keys are there
        if (rest < FTK) {
#pragma unroll
            for (int e = 0; e < 4; ++e)  // a row that is not there must not meet a numerator of 0 as an infinity
                if (e >= valid)
#pragma unroll
                    for (int h = 0; h < VH; ++h) v[e][h] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        if (tree) {  // nor must a node's infinities and NaN meet rows that do not see it: they are added at the end
            bool bad = false;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int h = 0; h < VH; ++h)
                    bad = bad || not_finite(v[e][h].x) || not_finite(v[e][h].y) || not_finite(v[e][h].z) || not_finite(v[e][h].w);
            if (__any(bad)) {
                dropped = true;
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int h = 0; h < VH; ++h) {
                        float4 &x = v[e][h];
                        x = make_float4(not_finite(x.x) ? 0.f : x.x, not_finite(x.y) ? 0.f : x.y, not_finite(x.z) ? 0.f : x.z,
                                        not_finite(x.w) ? 0.f : x.w);
                    }
            }
        }
        float p[RT][4];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const uint32_t seen = tree ? visible(rt, t - n_pref) >> (4 * lk) : 0xfu;
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[rt][e] = (s[rt][0][e] + s[rt][1][e]) + (s[rt][2][e] + s[rt][3][e]);
                if (e >= valid || !((seen >> e) & 1u)) p[rt][e] = -INFINITY;
                mx = fmaxf(mx, p[rt][e]);
            }
            if (__any(mx - m_run[rt] > kFloatRaise)) {  // (-inf - -inf is NaN: no)
                const float m_new = fmaxf(m_run[rt], keys_max(mx));
                const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[rt] - m_new);
                m_run[rt] = m_new;
                l_run[rt] *= alpha;
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[rt][h][j] *= alpha;
            }
            const float ref = m_run[rt] == -INFINITY ? 0.f : m_run[rt];  // no key with a score yet: numerators of zero
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[rt][e] = __builtin_amdgcn_exp2f(p[rt][e] - ref);
                sum += p[rt][e];
            }
            l_run[rt] += sum;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int h = 0; h < VH; ++h) {
                const float vv[4] = {v[e][h].x, v[e][h].y, v[e][h].z, v[e][h].w};
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        o[rt][h][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[j], p[rt][e], o[rt][h][j], 0, 0, 0);
            }
        if (t + FNW < n_all) load_v(t + FNW, v);
        if (++in_chain == kChain && t + FNW < n_all) {
            if (kept) add_kept();
            kept = true;
            in_chain = 0;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                put(rt);
                m_kept[rt] = m_run[rt];
#pragma unroll
                for (int h = 0; h < VH; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[rt][h][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    if (kept) add_kept();

    if (dropped) {
        for (int t = n_pref + (wave - n_pref % FNW + FNW) % FNW; t < n_all; t += FNW) {
            const int tt = t - n_pref;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                uint32_t word = visible(rt, tt) & 0xffffu;
                while (word) {
                    const float *row = vt + (int64_t)(tt * FTK + __builtin_ctz(word)) * a.vt_s[2] + 16 * lk;
                    word &= word - 1;
#pragma unroll
                    for (int h = 0; h < VH; ++h)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const float x = row[64 * h + 4 * e + j];
                                o[rt][h][j][e] += not_finite(x) ? x : 0.f;
                            }
                }
            }
        }
    }

    // ---- merge of the waves ---------------------------------------------------------------------------------
    constexpr int TPR = FNW * 64 / 16;  // threads per row
    const int n_active = n_all < FNW ? n_all : FNW;
    const int row = tid / TPR, piece = tid % TPR;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const float l_tot = keys_sum(l_run[rt]);
        if (lk == 0) ml_sh[(rt * 16 + li) * FNW + wave] = make_float2(m_run[rt], l_tot);
        if (busy) put(rt);
    }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int m = row0 + 16 * rt + row;
        if (m >= a.rows_kv || piece >= PPR) continue;
        float top = -INFINITY;
#pragma unroll
        for (int w = 0; w < FNW; ++w) top = fmaxf(top, ml_sh[(rt * 16 + row) * FNW + w].x);
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        float l_sum = 0.f;
#pragma unroll
        for (int w = 0; w < FNW; ++w) {
            if (w >= n_active) continue;
            const float2 ml = ml_sh[(rt * 16 + row) * FNW + w];
            const float scale = ml.x == -INFINITY ? (ml.y == 0.f ? 0.f : 1.f) : __builtin_amdgcn_exp2f(ml.x - top);
            const float4 x = o_sh[((rt * FNW + w) * 16 + row) * PPR + (piece ^ row)];
            l_sum = __builtin_fmaf(scale, ml.y, l_sum);
            sum.x = __builtin_fmaf(scale, x.x, sum.x);
            sum.y = __builtin_fmaf(scale, x.y, sum.y);
            sum.z = __builtin_fmaf(scale, x.z, sum.z);
            sum.w = __builtin_fmaf(scale, x.w, sum.w);
        }
        const float inv = l_sum == 0.f ? 0.f : 1.f / l_sum;  // no key with weight; NaN stays NaN
        const int hh = (int)divide(a.by_tree, (uint32_t)m), ti = m - hh * a.n_tree, hq = g * a.group + hh;
        const int64_t bh = (int64_t)b * a.n_q_heads + hq;
        const int64_t prow = a.o_parts ? bh * a.part_h + split * a.part_s + ti * a.part_t : bh * a.n_tree + ti;
        float *dst = a.o_parts ? a.o_parts + prow * D : a.out + b * a.o_s[0] + hq * a.o_s[1] + ti * a.o_s[2];
        if (l_sum == 0.f) sum = make_float4(0.f, 0.f, 0.f, 0.f);
        if (l_sum != 0.f || !a.split_tiles)  // (a piece without keys leaves its rows as they are)
            *(float4 *)(dst + 4 * piece) = make_float4(sum.x * inv, sum.y * inv, sum.z * inv, sum.w * inv);
        if (piece == 0) (a.o_parts ? a.lse_parts : a.lse)[prow] = l_sum == 0.f ? -INFINITY : (top + log2f(l_sum)) * kLn2;
    }
}

// Merge of the parts of a whole call, [query row, split]: a wavefront per query row, 64 / LG parts per load
// instruction, LG = D / 4 lanes a part.  A row whose part has a NaN is NaN.
struct FloatMergeArgs {
    const float *o_parts, *lse_parts;
    float *out, *lse;
    int64_t o_s[3];
    FastDiv by_tree, by_q_heads;
    int32_t n_splits, n_tree, n_q_heads, rows_total;
};

template <int D>
__global__ void __launch_bounds__(256) merge_float_kernel(FloatMergeArgs a)
{
    constexpr int LG = D / 4, GROUPS = kWave / LG, NL = 32 / GROUPS, PASS = 32;
    const int lane = threadIdx.x & (kWave - 1), group = lane / LG, sl = lane % LG;
    const int r = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + threadIdx.x / kWave);
    if (r >= a.rows_total) return;
    const int n = a.n_splits;
    const float *lses = a.lse_parts + (size_t)r * n;
    const float *rows = a.o_parts + (size_t)r * n * D + 4 * sl;
    float top = -INFINITY, wsum = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int p0 = 0; p0 < n; p0 += PASS) {
        float l[NL];
        float4 x[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            if (p0 + u * GROUPS >= n) break;  // wave-uniform
            const int part = p0 + u * GROUPS + group, at = part < n ? part : n - 1;
            l[u] = lses[at];
            x[u] = *(const float4 *)(rows + (size_t)at * D);
        }
        float mx = top;
#pragma unroll
        for (int u = 0; u < NL; ++u)
            if (p0 + u * GROUPS < n) mx = fmaxf(mx, l[u]);
#pragma unroll
        for (int off = LG; off < kWave; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
        const float keep = top == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((top - mx) * kLog2e);
        top = mx;
        wsum *= keep;
        acc.x *= keep;
        acc.y *= keep;
        acc.z *= keep;
        acc.w *= keep;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            if (p0 + u * GROUPS >= n) continue;
            if (p0 + u * GROUPS + group >= n) x[u] = make_float4(0.f, 0.f, 0.f, 0.f), l[u] = -INFINITY;  // (0 * inf)
            const float w = l[u] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((l[u] - top) * kLog2e);
            wsum += w;
            acc.x = __builtin_fmaf(w, x[u].x, acc.x);
            acc.y = __builtin_fmaf(w, x[u].y, acc.y);
            acc.z = __builtin_fmaf(w, x[u].z, acc.z);
            acc.w = __builtin_fmaf(w, x[u].w, acc.w);
        }
    }
#pragma unroll
    for (int off = LG; off < kWave; off <<= 1) {
        wsum += __shfl_xor(wsum, off, kWave);
        acc.x += __shfl_xor(acc.x, off, kWave);
        acc.y += __shfl_xor(acc.y, off, kWave);
        acc.z += __shfl_xor(acc.z, off, kWave);
        acc.w += __shfl_xor(acc.w, off, kWave);
    }
    if (group != 0) return;
    const int bh = (int)divide(a.by_tree, (uint32_t)r), i = r - bh * a.n_tree;
    const int b = (int)divide(a.by_q_heads, (uint32_t)bh), h = bh - b * a.n_q_heads;
    const float inv = wsum == 0.f ? 0.f : 1.f / wsum;
    *(float4 *)(a.out + b * a.o_s[0] + h * a.o_s[1] + i * a.o_s[2] + 4 * sl) =
        make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
    if (sl == 0) a.lse[r] = wsum == 0.f ? -INFINITY : top + log2f(wsum) * kLn2;
}

namespace {

FloatArgs float_args(const Problem &p, int n_splits)
{
    FloatArgs a{};
    a.prefix_lens = p.prefix_lens;
    a.q = (const float *)p.q;
    a.k_cache = (const float *)p.k_cache;
    a.v_cache = (const float *)p.v_cache;
    a.k_tree = (const float *)p.k_tree;
    a.v_tree = (const float *)p.v_tree;
    for (int i = 0; i < 3; ++i) {
        a.q_s[i] = p.q_stride[i];
        a.kc_s[i] = p.kc_stride[i], a.vc_s[i] = p.vc_stride[i];
        a.kt_s[i] = p.kt_stride[i], a.vt_s[i] = p.vt_stride[i];
    }
    a.prefix_len_all = p.prefix_len_all;
    a.max_prefix_len = p.max_prefix_len;
    a.n_tree = p.n_tree;
    a.rows_kv = p.group * p.n_tree;
    a.group = p.group;
    a.n_kv_heads = p.n_kv_heads;
    a.n_q_heads = p.n_q_heads;
    a.n_splits = n_splits;
    a.by_splits = FastDiv::of(n_splits);
    a.by_tree = FastDiv::of(p.n_tree);
    a.by_kv_heads = FastDiv::of(p.n_kv_heads);
    a.scale_log2 = p.scale_log2;
    return a;
}

template <int D, int RT> hipError_t launch_one(const FloatArgs &a, dim3 grid, dim3 block, hipStream_t stream)
{
    constexpr int lds_bytes = RT * FNW * 16 * (D * 4 + 8) + LS_MAX_TREE * 4 + (RT > 1 ? 16 * RT * D * 4 : 0);
    static std::atomic<uint64_t> allowed{0};
    if (const hipError_t e = allow_dynamic_lds((const void *)float_split_kernel<D, RT>, lds_bytes, allowed); e != hipSuccess) return e;
    hipLaunchKernelGGL((float_split_kernel<D, RT>), grid, block, lds_bytes, stream, a);
    return hipGetLastError();
}

hipError_t launch_float(FloatArgs a, int batch, int head_dim, int row_tiles, hipStream_t stream)
{
    const int64_t row_blocks = (a.rows_kv + 16 * row_tiles - 1) / (16 * row_tiles);
    a.by_row_blocks = FastDiv::of((uint32_t)row_blocks);
    const int64_t items = row_blocks * a.n_splits * batch * a.n_kv_heads;
    if (items >= 1ll << 32 || (head_dim != 64 && head_dim != 128)) return hipErrorInvalidValue;
    constexpr int64_t kMost = 1 << 22;  // workgroups per launch: HIP takes fewer than 2^32 threads
    for (int64_t first = 0; first < items; first += kMost) {
        a.first_item = (uint32_t)first;
        const dim3 grid((unsigned)(items - first < kMost ? items - first : kMost)), block(FNW * 64);
        const hipError_t e = head_dim == 128 ? (row_tiles == 2 ? launch_one<128, 2>(a, grid, block, stream) : launch_one<128, 1>(a, grid, block, stream))
                                             : (row_tiles == 2 ? launch_one<64, 2>(a, grid, block, stream) : launch_one<64, 1>(a, grid, block, stream));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_float_split(const Problem &p, int row_tiles, const WholeCall &w, hipStream_t stream)
{
    FloatArgs a = float_args(p, w.n_splits);
    a.parents = w.parents;
    a.err_flag = w.err_flag;
    if (w.in_parts) {
        a.o_parts = (float *)w.o_parts;
        a.lse_parts = w.lse_parts;
        a.part_h = (int64_t)p.n_tree * w.n_splits, a.part_s = 1, a.part_t = w.n_splits;
    } else {
        a.out = (float *)w.out;
        a.lse = w.lse;
        for (int i = 0; i < 3; ++i) a.o_s[i] = w.o_stride[i];
    }
    return launch_float(a, p.batch, p.head_dim, row_tiles, stream);
}

hipError_t launch_float_pieces(const Problem &p, const SplitPlan &plan, const Partials &out, hipStream_t stream)
{
    FloatArgs a = float_args(p, plan.n_splits);
    a.split_tiles = plan.split_len / FTK;
    const int64_t first = (int64_t)out.row(0, 0, p.n_tree, 0);
    a.o_parts = (float *)out.o + first * p.head_dim;
    a.lse_parts = out.lse + first;
    a.part_h = (int64_t)out.parts_stride * p.n_tree;
    a.part_s = out.row_major ? 1 : p.n_tree;
    a.part_t = out.row_major ? out.parts_stride : 1;
    return launch_float(a, p.batch, p.head_dim, a.rows_kv > 16 ? 2 : 1, stream);
}

hipError_t launch_merge_float(const Problem &p, const WholeCall &w, hipStream_t stream)
{
    FloatMergeArgs a{(const float *)w.o_parts, w.lse_parts, (float *)w.out, w.lse, {w.o_stride[0], w.o_stride[1], w.o_stride[2]},
                     FastDiv::of(p.n_tree), FastDiv::of(p.n_q_heads), w.n_splits, p.n_tree, p.n_q_heads,
                     p.batch * p.n_q_heads * p.n_tree};
    const dim3 grid((a.rows_total + 3) / 4), block(256);
    if (p.head_dim == 128) hipLaunchKernelGGL(merge_float_kernel<128>, grid, block, 0, stream, a);
    else if (p.head_dim == 64) hipLaunchKernelGGL(merge_float_kernel<64>, grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ls
