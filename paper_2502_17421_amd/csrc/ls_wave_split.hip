// Whole-path attention kernel whose waves split the keys: for calls with few query rows per KV head
// and for short caches (16-bit inputs).  Cached keys and tree keys go through the same loop, so the
// output of a workgroup that holds all keys of its rows is final and the call is one launch.
//
// Work decomposition.  A workgroup owns (sequence, KV head, 32 * RT query rows, key split); its
// eight waves all hold the same query rows and take the 32-key tiles of the split in turn.  A wave
// has a K stage and a V stage of LDS of its own, so the key loop needs no barrier: each wave runs at
// the pace its own tiles arrive.  At the end the eight partial results are merged through LDS in
// fp32, in fixed wave order, by the aggregation rule.  A split is a run of consecutive tiles, so the
// eight waves read 64 KB of neighbouring K rows and of V rows at a time (tiles dealt to the splits in
// turn instead: 59.4 against 54.9 us for 32 rows per KV head, 32 KV heads, 16k keys).
//
// What bounds it.  Short caches: the launch, then three dependent round trips (length, keys, output).  Long ones: with 32 or 64
// query rows a key tile of 16 KB costs 16 or 32 matrix instructions; 16k keys x 32 KV heads take 47.9 us, 5.6 TB/s of
// the 7.2 that a large read reaches, with the matrix cores busy for 0.08 of the cycles.  A wave requests the V rows of a
// tile once its K rows are there, and the next K rows once the V rows are, so one of its two stages is in flight at any time, 64 KB
// per workgroup; both in flight took as long, so that is not what holds it back, and the cause is not known.  (The kernel for
// many rows, ls_prefix_mfma.hip, shares tiles between its waves, which with few rows leaves waves without work.)
//
// Tree keys.  The tiles of the tree follow the cached tiles of the last split; the visibility of a
// row is a mask of its ancestors.  Up to 64 nodes it is built in registers, lane = node, by
// doubling the reach of every node (log2(depth) exchanges); larger trees walk the parent chain
// in LDS, once per tile.  The numerators of tree keys stay in fp32 (add_tree_product).
//
// More than one split: the rows leave as 16-bit partials for merge_parts_kernel, those of the split with
// the tree keys in fp32: the upper halves as a part row, the lower halves in the rows of `out` itself, which
// the merge reads before it overwrites them.
#include <type_traits>

#include "ls_internal.hpp"
#include "ls_mfma.hpp"

namespace ls {

namespace {

constexpr int TK = 32;            // keys per tile
constexpr int NW = 8;             // waves per workgroup
constexpr float kRaise = 8.f;     // the reference exponent is raised when a score exceeds it by 2^8

// A word that no kernel of the call writes, at a wave-uniform address: through the scalar cache, so that
// waiting for it does not wait for the copies in flight.
__device__ __forceinline__ int32_t scalar_load(const int32_t *p)
{
    return *(__attribute__((address_space(4))) const int32_t *)(uintptr_t)p;
}

// The mask word of tree tile `tt` for the chain of nodes starting at `node`, from its beginning.
__device__ __forceinline__ uint32_t chain_word(const int32_t *par, int node, int tt)
{
    while (node >= tt * 32 + 32) node = par[node];
    return take_chain_word(par, node, tt);
}

}  // namespace

// Arguments, in the order they are needed; all of them are fetched by one batch of scalar loads.  Strides in
// bytes.
struct WaveArgs {
    const int32_t *prefix_lens;
    const uint8_t *k_cache, *v_cache, *k_tree, *v_tree, *q;
    const int32_t *parents, *block_table;
    int64_t kc_b, kc_h, vc_b, vc_h, kt_b, kt_h, vt_b, vt_h;
    int64_t q_b, q_h, q_t;
    int32_t kc_r, vc_r, kt_r, vt_r;
    int32_t prefix_len_all, max_prefix_len, n_tree, rows_kv, group, n_kv_heads;
    FastDiv by_splits, by_tree, by_kv_heads, by_row_blocks;
    int32_t n_splits, bt_stride, page_shift, n_q_heads;
    float scale_log2;
    void *out;
    float *lse;
    int64_t o_b, o_h, o_t;
    void *o_parts;
    float *lse_parts;
    int32_t *err_flag;
};

// TREE: the call has tree keys; without them the code for them is not there (cross attention, 16 shapes 1.017 of the speed)
template <int D, bool F16, bool PAGED, int RT, bool TREE>
__global__ void __launch_bounds__(NW * 64, D == 64 && RT == 1 ? 4 : 2)
wave_split_kernel(WaveArgs a)
{
    constexpr int KSTEPS = D / 16;            // contraction steps of S^T = K Q^T
    constexpr int MT = D / 32;                // 32-row tiles of O^T along head_dim
    constexpr int CH = D / 8;                 // 16-byte chunks per row
    constexpr int ROWB = D * 2;               // bytes per row
    constexpr int TILEB = TK * ROWB;          // bytes per K (or V) tile
    constexpr int RPL = 64 / CH;              // rows one 64-lane copy covers
    constexpr int LOADS = TK / RPL;           // copies per tile and tensor
    constexpr uint32_t Q_OFF = NW * 2 * TILEB;                   // query rows (RT == 2 only)
    constexpr uint32_t PAR_OFF = Q_OFF + (RT > 1 ? RT * TILEB : 0);
    constexpr uint32_t ML_OFF = PAR_OFF + LS_MAX_TREE * 4;       // (m, l) of every wave and row
    typedef std::conditional_t<F16, half_t, uint16_t> T16;
    typedef __attribute__((address_space(3))) const uint4 *lds_u4;
    typedef __attribute__((address_space(3))) shortx4 *lds_s4;

    // Everything that the first requests need, in registers before anything is computed: left to itself the
    // compiler fetches the arguments a few at a time, each a round trip of its own.
    asm volatile("" ::"s"(a.prefix_lens), "s"(a.k_cache), "s"(a.v_cache), "s"(a.k_tree), "s"(a.v_tree), "s"(a.q), "s"(a.parents),
                 "s"(a.kc_b), "s"(a.kc_h), "s"(a.vc_b), "s"(a.vc_h), "s"(a.kt_b), "s"(a.kt_h), "s"(a.vt_b), "s"(a.vt_h),
                 "s"(a.q_b), "s"(a.q_h), "s"(a.q_t), "s"(a.kc_r), "s"(a.vc_r), "s"(a.kt_r), "s"(a.vt_r), "s"(a.n_tree),
                 "s"(a.rows_kv), "s"(a.by_splits.mul), "s"(a.by_tree.mul), "s"(a.by_kv_heads.mul), "s"(a.by_row_blocks.mul), "s"(a.n_splits));

    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x;
    const int hw_wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int li = lane & 31;
    const int lh = lane >> 5;

    // Workgroups are dealt to the eight XCDs in turn.  With several row blocks each XCD takes a run of consecutive work
    // items here (row block fastest, then split, then (sequence, KV head)), so that the row blocks that read the
    // same keys share an L2 (8 sequences x 8 KV heads, 160 query rows each, 1600 keys: 44.6 -> 26.2 us).  With one,
    // nothing is shared and runs would give whole sequences to an XCD, the longest one to a few of them.
    uint32_t item = blockIdx.x;
    if (a.by_row_blocks.d > 1) {
        const uint32_t xcd = blockIdx.x & 7u, per_xcd = gridDim.x >> 3, extra = gridDim.x & 7u;
        item = xcd * per_xcd + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
    }
    const uint32_t item_split = a.by_row_blocks.div(item);         // item / row blocks
    const uint32_t bz = a.by_splits.div(item_split);
    const int split = (int)(item_split - bz * (uint32_t)a.n_splits);
    const int b = (int)a.by_kv_heads.div(bz);
    const int g = (int)bz - b * a.n_kv_heads;
    const int rows_kv = a.rows_kv;
    const int row_block = (int)(item - item_split * a.by_row_blocks.d);
    const int row0 = row_block * (32 * RT);  // first query row (of the KV head) of this workgroup
    const uint32_t smem_off = lds_offset(smem);

    // ---- this split's tiles: cached ones, then (last split) those of the tree --------------------
    int plen = a.prefix_lens ? scalar_load(a.prefix_lens + b) : a.prefix_len_all;
    plen = plen < 0 ? 0 : (plen > a.max_prefix_len ? a.max_prefix_len : plen);
    const int n_splits = a.n_splits;
    const int all_pref = (plen + TK - 1) / TK;
    const int tree_tiles = TREE ? (a.n_tree + TK - 1) / TK : 0;
    const bool last_split = split == n_splits - 1;
    const bool has_tree = TREE && last_split;
    const int per_split = (int)a.by_splits.div((uint32_t)(all_pref + tree_tiles + n_splits - 1));
    int t_lo = split * per_split;
    t_lo = t_lo < all_pref ? t_lo : all_pref;
    int t_hi = last_split ? all_pref : t_lo + per_split;
    t_hi = t_hi < all_pref ? t_hi : all_pref;
    const int n_pref = t_hi - t_lo;
    const int n_all = n_pref + (has_tree ? tree_tiles : 0);
    // Tile t of the split belongs to wave t % NW, so a tree tile, which takes about as long as two cached ones (its mask, three
    // products, K and V one after the other), may fall to any wave.  The hardware starts waves 0 to 3 first, and serves
    // them first on the SIMD that each shares with one of 4 to 7; so where the tree tiles fall to the latter the halves change
    // places.  Which tiles are added up together, and in which order, stays as it is.  Not where the tree tiles run on into wave 0:
    // those waves have one more cached tile than the others (8 sequences x 290 rows 22.4 / 25.3 us with the exchange).
    // Against no exchange, 8 KV heads x 32 rows: 640 keys 10.4 -> 8.9 us, 926 keys 11.5 -> 10.0, 1500 keys 14.6 -> 13.4;
    // 174 shapes 0.969 of the time, worst 1.024.  Tree tiles dealt to the first waves, which leave out cached ones: 640 keys 9.1, but 1100
    // 10.6 / 11.8 and in pages 12.3 / 14.1, and the rounding error grew by up to 4 %: fewer waves start from a row's largest score.
    const int wave = hw_wave ^ (TREE && (n_pref & (NW / 2)) && (n_pref & (NW - 1)) + n_all - n_pref <= NW ? NW / 2 : 0);
    const uint32_t k_stage = smem_off + wave * 2 * TILEB;  // the V stage follows
    auto tile_row = [&](int t) __attribute__((always_inline)) { return (t_lo + t) * TK; };  // of cached tile t of the split

    const uint8_t *kc = uniform_ptr(a.k_cache + (PAGED ? 0 : b * a.kc_b) + g * a.kc_h);
    const uint8_t *vc = uniform_ptr(a.v_cache + (PAGED ? 0 : b * a.vc_b) + g * a.vc_h);
    const uint8_t *kt = uniform_ptr(a.k_tree + b * a.kt_b + g * a.kt_h);
    const uint8_t *vt = uniform_ptr(a.v_tree + b * a.vt_b + g * a.vt_h);
    const int ld_row = lane / CH, ld_pos = lane % CH;
    // chunk a lane fetches: its LDS position under the row's swizzle.  Copy j covers rows j*RPL ..; for
    // head_dim 128 (four rows per copy) the K swizzle of those rows is that of rows 0..3 with 4*(j%4) added
    const uint32_t k_chunk = (uint32_t)(ld_pos ^ ld_row), v_chunk = (uint32_t)(ld_pos ^ (vswz(ld_row) & (CH - 1)));
    const int page_rows_mask = (1 << a.page_shift) - 1;
    const int32_t *tab = PAGED ? a.block_table + (int64_t)b * a.bt_stride : nullptr;

    // Paged cache: the pages of rows 0..15 and 16..31 of cached tile t (equal for pages of 32 rows and more)
    auto pages_of = [&](int t) __attribute__((always_inline)) {
        int2 ids = make_int2(0, 0);
        if constexpr (PAGED) {
            const int r0 = tile_row(t), r1 = r0 + 16;
            if (t < n_pref) {
                ids.x = scalar_load(tab + (r0 >> a.page_shift));
                ids.y = scalar_load(tab + ((r1 < plen ? r1 : plen - 1) >> a.page_shift));
            }
        }
        return ids;
    };
    // all LOADS copies of tile t of this split (K or V, wave-uniform) into this wave's stage
    auto request = [&](bool is_v, int t, int2 pages) __attribute__((always_inline)) {
        const uint32_t dst = __builtin_amdgcn_readfirstlane(k_stage + (is_v ? TILEB : 0));
        const bool tree = t >= n_pref;
        const int first = tree ? (t - n_pref) * TK : tile_row(t);   // first row of the tile
        const int last = (tree ? a.n_tree : plen) - 1 - first;      // last valid row, relative
        const int32_t rb_cache = is_v ? a.vc_r : a.kc_r, rb_tree = is_v ? a.vt_r : a.kt_r;
        const int32_t rb = tree ? rb_tree : rb_cache;
        const uint8_t *base = is_v ? (tree ? vt : vc) : (tree ? kt : kc);
        const uint32_t chunk = (is_v ? v_chunk : k_chunk) * 16;
        // copy j's chunk: K rows at head_dim 128 add 4*(j%4) to the swizzle
        auto chunk_of = [&](int j) __attribute__((always_inline)) {
            return RPL >= CH ? chunk : chunk ^ (uint32_t)(is_v ? 0 : ((j * RPL) & (CH - 1)) * 16);
        };
        if (!PAGED || tree) {
            base += (int64_t)first * rb;
            if (last >= TK - 1) {
                const uint32_t off = (uint32_t)(ld_row * rb);
#pragma unroll
                for (int j = 0; j < LOADS; ++j) {
                    copy_to_lds(base, off + chunk_of(j), dst + j * RPL * ROWB);
                    base += RPL * rb;
                }
            } else {  // rows past the end repeat the last one; their scores are masked
#pragma unroll 1
                for (int j = 0; j < LOADS; ++j) {
                    const int row = j * RPL + ld_row;
                    copy_to_lds(base, (uint32_t)((row < last ? row : last) * rb) + chunk_of(j), dst + j * RPL * ROWB);
                }
            }
        } else {
            const int64_t page_bytes = is_v ? a.vc_b : a.kc_b;
            // a copy covers RPL consecutive rows, which never straddle a page; rows past the end
            // repeat the last one, fetched through that row's own group
            const int last_group = last & ~(RPL - 1);
#pragma unroll
            for (int j = 0; j < LOADS; ++j) {
                const int src0 = j * RPL < last_group ? j * RPL : last_group;
                int src = src0 + ld_row;
                src = src < last ? src : last;
                const int64_t page = src0 < 16 ? pages.x : pages.y;
                copy_to_lds(base + page * page_bytes + (int64_t)((first + src0) & page_rows_mask) * rb,
                            (uint32_t)((src - src0) * rb) + chunk_of(j), dst + j * RPL * ROWB);
            }
        }
    };
    const bool busy = wave < n_all;
    // Requests go out in the order their data is needed and can be addressed: first keys, query rows (RT == 1:
    // to registers; RT == 2: to LDS, eight rows per wave, in the K tiles' swizzled layout), parents of the
    // tree (one node per lane), first values.  Loads return in order, so waiting for all but the values'
    // copies waits for everything before them.
    int2 pages = make_int2(0, 0);
    if (busy) {
        pages = pages_of(wave);
        request(false, wave, pages);
    }
    auto row_of = [&](int m) __attribute__((always_inline)) { return m < rows_kv ? m : rows_kv - 1; };  // rows past the end repeat the last
    auto q_row_ptr = [&](int m) __attribute__((always_inline)) {
        const int hh = (int)a.by_tree.div((uint32_t)m), ti = m - hh * a.n_tree;
        return (const uint16_t *)(a.q + b * a.q_b + (g * a.group + hh) * a.q_h + ti * a.q_t);
    };
    u32x4 q_raw[RT == 1 ? KSTEPS : 1];
    if constexpr (RT == 1) {
        const uint16_t *q_ptr = q_row_ptr(row_of(row0 + li));
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
            asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(q_raw[kk]) : "v"(q_ptr + kk * 16 + lh * 8) : "memory");
    } else {
        constexpr int COPIES = 32 * RT / NW / RPL;  // of RPL rows each
#pragma unroll
        for (int j = 0; j < COPIES; ++j) {
            const int row = wave * (32 * RT / NW) + j * RPL + ld_row;
            const uint16_t *src = q_row_ptr(row_of(row0 + row)) + (ld_pos ^ (row & (CH - 1))) * 8;
            copy_row_to_lds(src, __builtin_amdgcn_readfirstlane(smem_off + Q_OFF + (wave * (32 * RT / NW) + j * RPL) * ROWB));
        }
    }
    int32_t par_reg = 0;
    if constexpr (TREE) {  // loaded on every path, from a valid address, so that the register is written by one instruction
        const int32_t *src = has_tree ? a.parents + (int64_t)b * a.n_tree + (lane < a.n_tree ? lane : 0) : (const int32_t *)a.q;
        asm volatile("global_load_dword %0, %1, off" : "=v"(par_reg) : "v"(src) : "memory");
    }
    if (busy) request(true, wave, pages);
    int2 pages_next = pages_of(wave + NW);
    if (busy) wait_vmem<LOADS>();
    else wait_vmem<0>();
    bf16x8 q_reg[RT == 1 ? KSTEPS : 1];
    if constexpr (RT == 1) {
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            asm volatile("" : "+v"(q_raw[kk]));  // orders every use below after the wait above
            q_reg[kk] = __builtin_bit_cast(bf16x8, q_raw[kk]);
        }
    } else {
        asm volatile("s_barrier" ::: "memory");  // every wave's query rows are in LDS
    }
    if constexpr (TREE) asm volatile("" : "+v"(par_reg));

    // ---- tree mask ---------------------------------------------------------------------------------
    int32_t *par_lds = (int32_t *)(smem + PAR_OFF);  // parents; up to 64 nodes: the mask of every node instead
    bool bad_parent = false;
    const bool tree_wave = has_tree && busy && n_all > n_pref && wave + ((n_all - 1 - wave) / NW) * NW >= n_pref;
    if (TREE && tree_wave) {  // wave-uniform
        if (a.n_tree <= 64) {
            int anc = par_reg;
            if (lane < a.n_tree) {
                if (anc < -1 || anc >= lane) {  // not a forest in topological order: treat the node as a root
                    bad_parent = true;
                    anc = -1;
                }
            } else {
                anc = -1;
            }
            const uint2 mask = ancestor_mask(anc, lane);
            ((uint2 *)par_lds)[lane] = mask;  // (every wave that needs it writes the same values)
        } else {
            // every wave that needs the array writes all of it: the waves write the same values
            for (int i = lane; i < a.n_tree; i += 64) {
                int pa = a.parents[(size_t)b * a.n_tree + i];
                if (pa < -1 || pa >= i) {
                    bad_parent = true;
                    pa = -1;
                }
                par_lds[i] = pa;
            }
        }
        // the wave of the first tree tile reports
        if (n_pref % NW == wave && g == 0 && row_block == 0) {
            const bool any_bad = __any(bad_parent);
            if (lane == 0 && a.err_flag) a.err_flag[b] = any_bad ? 1 : 0;
        }
    }

    // ---- key loop ------------------------------------------------------------------------------------
    floatx16 o_acc[RT][MT];
    float m_run[RT], l_run[RT];  // reference exponent (raw scores); sum of the numerators of this lane's keys
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m_run[rt] = -INFINITY;
        l_run[rt] = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o_acc[rt][mt][e] = 0.f;
    }
    const float c = a.scale_log2;
    // per-lane LDS addresses of the operand fragments (see ls_prefix_mfma.hip: fragment f is one XOR away)
    const uint32_t k_off0 = k_stage + li * ROWB + ((lh ^ (li & (CH - 1))) * 16);
    const uint32_t q_off0 = smem_off + Q_OFF + li * ROWB + ((lh ^ (li & (CH - 1))) * 16);
    const int tr_s = lane & 15;
    const int tr_row = 4 * lh + (tr_s >> 2);
    const int tr_dchunk = 2 * ((lane >> 4) & 1) + ((tr_s & 3) >> 1);
    const uint32_t v_off0 = k_stage + TILEB + tr_row * ROWB + ((tr_dchunk ^ (vswz(tr_row) & (CH - 1))) * 16) + (tr_s & 1) * 8;

    auto read_k_tile = [&](bf16x8 (&frag)[KSTEPS]) __attribute__((always_inline)) {
        uint32_t off = k_off0;
        asm volatile("" : "+v"(off));  // the fragments' addresses are formed here, not kept over the loop
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
            frag[kk] = __builtin_bit_cast(bf16x8, *(lds_u4)(uintptr_t)(off ^ (uint32_t)(kk << 5)));
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) asm volatile("" : "+v"(frag[kk]));  // in registers: the stage is free
    };
    auto read_v = [&](uint32_t off, int f) __attribute__((always_inline)) {  // f = 16-key half * MT + d tile
        const uint32_t a = (off ^ (uint32_t)((f % MT) << 6)) + ((f / MT) * 16) * ROWB;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)a);
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(uintptr_t)(a + 8 * ROWB));
        const uint2 lo2 = __builtin_bit_cast(uint2, lo), hi2 = __builtin_bit_cast(uint2, hi);
        return __builtin_bit_cast(bf16x8, make_uint4(lo2.x, lo2.y, hi2.x, hi2.y));
    };
    auto read_v_tile = [&](bf16x8 (&frag)[KSTEPS]) __attribute__((always_inline)) {
        uint32_t off = v_off0;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int f = 0; f < KSTEPS; ++f) frag[f] = read_v(off, f);
#pragma unroll
        for (int f = 0; f < KSTEPS; ++f) asm volatile("" : "+v"(frag[f]));
    };
    auto scores = [&](const bf16x8 (&frag)[KSTEPS], int rt, floatx16 &s) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
        uint32_t off = q_off0 + rt * TILEB;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            bf16x8 q;
            if constexpr (RT == 1) q = q_reg[kk];
            else q = __builtin_bit_cast(bf16x8, *(lds_u4)(uintptr_t)(off ^ (uint32_t)(kk << 5)));
            s = mfma32<F16>(frag[kk], q, s);
        }
    };
    // raises the reference exponent of row tile rt where the scores are more than `lazy` powers of two above it
    // (start: nothing has been accumulated yet; up: the sums so far are multiplied by this as well)
    auto raise = [&](int rt, const floatx16 &s, bool start, float lazy, float up) __attribute__((always_inline)) {
        float mx = s[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
        mx = half_max(mx);
        if (start) {
            m_run[rt] = mx;
        } else if (up != 1.f || __any((mx - m_run[rt]) * c > lazy)) {  // also while m_run is -inf
            const float m_new = fmaxf(m_run[rt], mx);
            const float alpha = (m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((m_run[rt] - m_new) * c)) * up;
            m_run[rt] = m_new;
            l_run[rt] *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int e = 0; e < 16; ++e) o_acc[rt][mt][e] *= alpha;
        }
    };
    auto add_product = [&](const bf16x8 (&frag)[KSTEPS], int rt, const uint32_t (&pp)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < KSTEPS; ++f) {
            const uint32_t *q = pp + 4 * (f / MT);
            o_acc[rt][f % MT] = mfma32<F16>(frag[f], __builtin_bit_cast(bf16x8, make_uint4(q[0], q[1], q[2], q[3])),
                                            o_acc[rt][f % MT]);
        }
    };

    bool not_finite = false;  // wave-uniform: infinities or NaN among the values of this wave's tree tiles
    int t = wave;
    for (; t < n_pref; t += NW) {  // cached keys
        const bool more = t + NW < n_all;
        bf16x8 frag[KSTEPS];
        uint32_t pp[RT][8];  // numerators in the operand type
        if (t == wave) {
            wait_vmem<LOADS>();  // the K rows; the V rows are the LOADS copies behind them
        } else {
            wait_vmem<0>();
            request(true, t, pages);
        }
        read_k_tile(frag);
        const int valid = plen - tile_row(t);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            floatx16 s;
            scores(frag, rt, s);
            if (valid < TK) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e >> 2) + 4 * lh + (e & 3) >= valid) s[e] = -INFINITY;
            }
            raise(rt, s, t == wave, kRaise, 1.f);
            // a row all of whose scores so far are -inf has the reference -inf: its numerators are zeros
            const float mc = m_run[rt] == -INFINITY ? 0.f : m_run[rt] * c;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c, -mc));
                const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], c, -mc));
                sum += p0 + p1;
                pp[rt][e >> 1] = pack16<F16>(p0, p1);
            }
            l_run[rt] += sum;
        }
        wait_vmem<0>();  // the V rows of tile t
        pages = pages_next;
        if (more) request(false, t + NW, pages);
        pages_next = pages_of(t + 2 * NW);
        read_v_tile(frag);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) add_product(frag, rt, pp[rt]);
    }
    auto visible = [&](int rt, int tt) __attribute__((always_inline)) {  // nodes of tree tile tt that this lane's row sees
        const int m = row_of(row0 + rt * 32 + li);
        const int node = m - (int)a.by_tree.div((uint32_t)m) * a.n_tree;
        return a.n_tree > 64 ? chain_word(par_lds, node, tt) : (uint32_t)par_lds[2 * node + tt];
    };
    for (; TREE && t < n_all; t += NW) {  // tree keys; one row tile after the other
        if (t != wave) request(true, t, pages);
        wait_vmem<0>();
        const int tt = t - n_pref;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            bf16x8 frag[KSTEPS];
            read_k_tile(frag);
            floatx16 s;
            scores(frag, rt, s);
            const uint32_t seen = visible(rt, tt) >> (4 * lh);
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (!((seen >> (8 * (e >> 2) + (e & 3))) & 1u)) s[e] = -INFINITY;
            raise(rt, s, t == wave, F16 ? 0.f : kRaise, t - NW < n_pref ? kTreeUp<F16> : 1.f);
            uint32_t parts[kTreeParts<F16>][8];
            l_run[rt] += tree_numerators<F16>(s, c, m_run[rt], parts);
            __builtin_amdgcn_sched_barrier(0);  // the values are not read early: no registers to spare
            read_v_tile(frag);
            not_finite |= drop_not_finite<F16>(frag);
            add_tree_product<F16>(o_acc[rt], frag, parts);
        }
        if (t + NW < n_all) request(false, t + NW, pages);
    }

    if (TREE && not_finite) {
        for (t = n_pref + (wave - n_pref) % NW; t < n_all; t += NW) {
            const int tt = t - n_pref;
            if (tt < 0) continue;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                uint32_t word = visible(rt, tt);
                while (word) {
                    const int node = tt * 32 + __builtin_ctz(word);
                    word &= word - 1;
                    add_not_finite<F16>(o_acc[rt], vt + (int64_t)node * a.vt_r, lh);
                }
            }
        }
    }

    // ---- merge of the waves, in fp32, through the stages (each wave its own: nothing reads them any more)
    constexpr int CPR = D / 4;                // 16-byte pieces (4 floats) per output row
    constexpr int TPR = NW * 64 / 32;         // threads per row
    constexpr int PASSES = CPR / TPR;         // pieces per thread
    float2 *ml = (float2 *)(smem + ML_OFF);   // (m, l) [row][wave]
    const int n_active = n_all < NW ? n_all : NW;
    const int row = tid / TPR;                // the row this thread finishes
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        if (rt) __syncthreads();  // the rows of the previous tile have been read
        const float l_tot = half_sum(l_run[rt]);
        if (lh == 0) ml[li * NW + wave] = make_float2(m_run[rt], l_tot);
        if (busy) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const int piece = (8 * mt + 2 * rg + lh) ^ (li & (CPR - 1));
                    *(float4 *)(smem + wave * 2 * TILEB + li * (D * 4) + piece * 16) =
                        make_float4(o_acc[rt][mt][4 * rg], o_acc[rt][mt][4 * rg + 1], o_acc[rt][mt][4 * rg + 2],
                                    o_acc[rt][mt][4 * rg + 3]);
                }
        }
        const int m = row0 + rt * 32 + row;
        const int hh = (int)a.by_tree.div((uint32_t)m), ti = m - hh * a.n_tree, hq = g * a.group + hh;
        const size_t row_id = ((size_t)b * a.n_q_heads + hq) * a.n_tree + ti;
        const bool final_row = n_splits == 1;
        const size_t prow = row_id * n_splits + split;
        T16 *orow = (T16 *)((uint8_t *)a.out + b * a.o_b + hq * a.o_h + ti * a.o_t);
        T16 *dst = final_row ? orow : (T16 *)a.o_parts + prow * D;
        __syncthreads();
        float2 s[NW];
        float4 v[PASSES][NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) s[k] = ml[row * NW + k];
#pragma unroll
        for (int k = 0; k < NW; ++k)
            if (k < n_active)  // wave-uniform
#pragma unroll
                for (int u = 0; u < PASSES; ++u)
                    v[u][k] = *(const float4 *)(smem + k * 2 * TILEB + row * (D * 4) +
                                                (((tid % TPR + u * TPR) ^ (row & (CPR - 1))) * 16));
        float top = s[0].x;
#pragma unroll
        for (int k = 1; k < NW; ++k) top = fmaxf(top, s[k].x);
        float o[PASSES][4], l_sum = 0.f;
#pragma unroll
        for (int u = 0; u < PASSES; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[u][i] = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (k >= n_active) continue;
            const bool tree = TREE && ((k - n_pref) & (NW - 1)) < n_all - n_pref;  // this wave had tree tiles: its sums are lifted
            const float scale = s[k].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((s[k].x - top) * c) * (tree ? kTreeDown<F16> : 1.f);
            l_sum += scale * s[k].y;
#pragma unroll
            for (int u = 0; u < PASSES; ++u) {
                o[u][0] += scale * v[u][k].x;
                o[u][1] += scale * v[u][k].y;
                o[u][2] += scale * v[u][k].z;
                o[u][3] += scale * v[u][k].w;
            }
        }
        const float inv = l_sum == 0.f ? 0.f : 1.f / l_sum;  // no key with weight; NaN stays NaN, in the LSE too
        if (m >= rows_kv) continue;
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            const int col = (tid % TPR + u * TPR) * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[u][i] *= inv;
            if (has_tree && !final_row) {  // fp32, in two halves
                *(uint2 *)(dst + col) = make_uint2(upper_halves(o[u][0], o[u][1]), upper_halves(o[u][2], o[u][3]));
                *(uint2 *)(orow + col) = make_uint2(lower_halves(o[u][0], o[u][1]), lower_halves(o[u][2], o[u][3]));
            } else {
                *(uint2 *)(dst + col) = make_uint2(pack16<F16>(o[u][0], o[u][1]), pack16<F16>(o[u][2], o[u][3]));
            }
        }
        if (tid % TPR == 0) {
            const float lse = l_sum == 0.f ? -INFINITY : (top * c + log2f(l_sum)) * kLn2;
            (final_row ? a.lse : a.lse_parts)[prow] = lse;
        }
    }
}

namespace {

template <int D, bool F16, bool PAGED, int RT, bool TREE>
hipError_t launch_one(WaveArgs a, int batch, hipStream_t stream)
{
    constexpr int lds_bytes = NW * 2 * TK * D * 2 + (RT > 1 ? RT * TK * D * 2 : 0) + LS_MAX_TREE * 4 + NW * 32 * 8;
    static_assert(lds_bytes <= 160 * 1024, "the stages exceed the 160 KB of a compute unit");
    auto kernel = wave_split_kernel<D, F16, PAGED, RT, TREE>;
    static std::atomic<uint64_t> allowed{0};
    if (const hipError_t e = allow_dynamic_lds((const void *)kernel, lds_bytes, allowed); e != hipSuccess) return e;
    const int64_t row_blocks = (a.rows_kv + 32 * RT - 1) / (32 * RT);
    const int64_t items = row_blocks * a.n_splits * batch * a.n_kv_heads;
    // (the bound keeps the kernel's divisions exact)
    if (items * (row_blocks > a.n_splits ? row_blocks : a.n_splits) >= (1ll << 32)) return hipErrorInvalidValue;
    a.by_row_blocks = FastDiv::of((uint32_t)row_blocks);
    hipLaunchKernelGGL(kernel, dim3((unsigned)items), dim3(NW * 64), lds_bytes, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_wave_split(const Problem &p, int dtype, int row_tiles, const WholeCall &w, hipStream_t stream)
{
    if (dtype == LS_F32) return launch_float_split(p, row_tiles, w, stream);
    const bool f16 = dtype == LS_F16;
    const bool paged = p.block_table != nullptr;
    WaveArgs a{};
    a.prefix_lens = p.prefix_lens;
    a.k_cache = (const uint8_t *)p.k_cache;
    a.v_cache = (const uint8_t *)p.v_cache;
    a.k_tree = (const uint8_t *)p.k_tree;
    a.v_tree = (const uint8_t *)p.v_tree;
    a.q = (const uint8_t *)p.q;
    a.parents = w.parents;
    a.block_table = p.block_table;
    a.kc_b = 2 * p.kc_stride[0], a.kc_h = 2 * p.kc_stride[1], a.kc_r = (int32_t)(2 * p.kc_stride[2]);
    a.vc_b = 2 * p.vc_stride[0], a.vc_h = 2 * p.vc_stride[1], a.vc_r = (int32_t)(2 * p.vc_stride[2]);
    a.kt_b = 2 * p.kt_stride[0], a.kt_h = 2 * p.kt_stride[1], a.kt_r = (int32_t)(2 * p.kt_stride[2]);
    a.vt_b = 2 * p.vt_stride[0], a.vt_h = 2 * p.vt_stride[1], a.vt_r = (int32_t)(2 * p.vt_stride[2]);
    a.q_b = 2 * p.q_stride[0], a.q_h = 2 * p.q_stride[1], a.q_t = 2 * p.q_stride[2];
    a.o_b = 2 * w.o_stride[0], a.o_h = 2 * w.o_stride[1], a.o_t = 2 * w.o_stride[2];
    a.prefix_len_all = p.prefix_len_all;
    a.max_prefix_len = p.max_prefix_len;
    a.n_tree = p.n_tree;
    a.rows_kv = p.group * p.n_tree;
    a.group = p.group;
    a.n_kv_heads = p.n_kv_heads;
    a.n_q_heads = p.n_q_heads;
    a.by_splits = w.by_splits;
    a.by_tree = w.by_tree;
    a.by_kv_heads = w.by_kv_heads;
    a.n_splits = w.n_splits;
    a.bt_stride = p.bt_stride;
    a.page_shift = p.page_shift;
    a.scale_log2 = p.scale_log2;
    a.out = w.out;
    a.lse = w.lse;
    a.o_parts = w.o_parts;
    a.lse_parts = w.lse_parts;
    a.err_flag = w.err_flag;
#define LS_WS_CASE3(DD, RR, TT)                                                                                             \
    (paged ? (f16 ? launch_one<DD, true, true, RR, TT>(a, p.batch, stream) : launch_one<DD, false, true, RR, TT>(a, p.batch, stream)) \
           : (f16 ? launch_one<DD, true, false, RR, TT>(a, p.batch, stream) : launch_one<DD, false, false, RR, TT>(a, p.batch, stream)))
#define LS_WS_CASE2(DD, RR) (w.parents ? LS_WS_CASE3(DD, RR, true) : LS_WS_CASE3(DD, RR, false))
#define LS_WS_CASE(DD) (row_tiles == 1 ? LS_WS_CASE2(DD, 1) : LS_WS_CASE2(DD, 2))
    if (p.head_dim == 128) return LS_WS_CASE(128);
    if (p.head_dim == 64) return LS_WS_CASE(64);
#undef LS_WS_CASE
#undef LS_WS_CASE2
#undef LS_WS_CASE3
    return hipErrorInvalidValue;
}

}  // namespace ls
