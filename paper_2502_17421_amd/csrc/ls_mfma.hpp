// Matrix-core building blocks shared by the cached-key kernels (16-bit inputs, gfx950): operand types,
// the 32x32x16 product, packs, half-wave exchanges, HBM -> LDS copies and their waits, the V swizzle.
//
// MFMA layouts used (v_mfma_f32_32x32x16_bf16 / _f16, A is 32xK, B is Kx32, K = 16):
//   A: lane l holds row l % 32, contraction indices 8*(l/32) .. 8*(l/32)+7
//   B: lane l holds column l % 32, same contraction indices
//   C/D: lane l, register r holds row 8*(r/4) + 4*(l/32) + r%4, column l % 32
// Only the C/D layout and the pairing of contraction slices between A and B matter.
// ds_read_b64_tr_b16, per block of 16 lanes: lane L receives element L%4 of the four
// 8-byte pieces addressed by lanes L/4, L/4+4, L/4+8, L/4+12 of its block.
#pragma once

#include "ls_internal.hpp"

namespace ls {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));  // also carries eight IEEE halves as bit patterns
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool F16> __device__ __forceinline__ floatx16 mfma32(bf16x8 a, bf16x8 b, floatx16 c)
{
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c,
                                                      0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// two floats to one register of the operand type, round to nearest even
template <bool F16> __device__ __forceinline__ uint32_t pack16(float lo, float hi)
{
    floatx2 f = {lo, hi};
    if constexpr (F16) {
        typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, halfx2));
    } else {
        bf16x2 b = __builtin_convertvector(f, bf16x2);
        return __builtin_bit_cast(uint32_t, b);
    }
}
// the softmax numerators: one instruction per pair in either type (halves round toward zero,
// a bias of 2^-12 of the value that the fp32 row sums do not share; far below the output's
// own rounding)
template <bool F16> __device__ __forceinline__ uint32_t pack_numerators(float lo, float hi)
{
    if constexpr (F16) return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
    else return pack16<false>(lo, hi);
}

// max / sum across the two 32-lane halves of the wave (lane l with lane l ^ 32)
__device__ __forceinline__ float half_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One 64-lane HBM -> LDS copy: lane l moves 16 bytes from base + voff[l] to LDS byte
// lds_base + 16*l (base and lds_base wave-uniform; lds_base goes through M0).  Written as
// inline assembly so that the compiler does not serialise later LDS reads behind all copies
// still in flight; the kernel orders reads after copies itself with wait_vmem + a barrier.
// M0 cannot be named as clobbered (the compiler ignores reserved registers in a clobber list and
// warns); it writes M0 itself only for instructions these kernels do not contain, which the test
// suite checks on the generated assembly (every M0 access belongs to one of these copies).
__device__ __forceinline__ void copy_to_lds(const uint8_t *base, uint32_t voff, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_base), "v"(voff), "s"(base)
                 : "memory");
}

// The same with an address per lane.
__device__ __forceinline__ void copy_row_to_lds(const void *src, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"(src) : "memory");
}

__device__ __forceinline__ const uint8_t *uniform_ptr(const uint8_t *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const uint8_t *)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ uint32_t lds_offset(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

template <int N> __device__ __forceinline__ void wait_vmem()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// V swizzle: row r of a V tile stores its 16-byte chunk c at position c ^ vswz(r).  Rows
// r, r+1, r+2, r+3 then put the 32-byte pieces one transpose read touches on distinct banks.
__device__ __forceinline__ int vswz(int row)
{
    const int k = row & 3;
    return (((k >> 1) << 2) | ((k & 1) << 1) | (k >> 1)) << 1;
}

// the two values of a packed pair
template <bool F16> __device__ __forceinline__ float low16(uint32_t u)
{
    return F16 ? half_to_float((uint16_t)u) : __uint_as_float(u << 16);
}
template <bool F16> __device__ __forceinline__ float high16(uint32_t u)
{
    return F16 ? half_to_float((uint16_t)(u >> 16)) : __uint_as_float(u & 0xffff0000u);
}

// The row of a split that holds tree keys leaves in fp32: the upper halves of its values in its row of the parts,
// the lower halves in the row of `out` (merge_parts_kernel joins them).
__device__ __forceinline__ uint32_t upper_halves(float a, float b)
{
    return __float_as_uint(a) >> 16 | (__float_as_uint(b) & 0xffff0000u);
}
__device__ __forceinline__ uint32_t lower_halves(float a, float b)
{
    return (__float_as_uint(a) & 0xffffu) | __float_as_uint(b) << 16;
}

// ---- tree keys on the matrix cores ------------------------------------------------------------
// A tree tile holds 32 nodes; a row sees a node when it is an ancestor of the row's own node or that
// node itself.  Numerators of tree keys stay in fp32 (add_tree_product), as in the tail kernel: the few tree
// keys may carry most of a row's weight.

// Ancestors of node `lane` (itself included) as a 64-bit mask, for trees of at most 64 nodes: every
// round doubles the reach of every node.  anc: the node's parent, valid or -1; all 64 lanes active.
__device__ __forceinline__ uint2 ancestor_mask(int anc, int lane)
{
    uint32_t lo = lane < 32 ? 1u << lane : 0u, hi = lane < 32 ? 0u : 1u << (lane - 32);
    while (__any(anc >= 0)) {
        const int src = (anc < 0 ? lane : anc) * 4;
        const uint32_t lo2 = __builtin_amdgcn_ds_bpermute(src, lo), hi2 = __builtin_amdgcn_ds_bpermute(src, hi);
        const int anc2 = __builtin_amdgcn_ds_bpermute(src, anc);
        if (anc >= 0) {
            lo |= lo2;
            hi |= hi2;
            anc = anc2;
        }
    }
    return make_uint2(lo, hi);
}

// The mask word of tree tile `tt` (bit k: node 32*tt + k) of a chain walked in LDS (entries -1 or
// smaller than their index): takes the nodes of that tile off the chain.  Tiles are visited from the
// last one down, as the chain does.
__device__ __forceinline__ uint32_t take_chain_word(const int32_t *par, int &node, int tt)
{
    uint32_t bits = 0;
    while (node >= tt * 32) {
        bits |= 1u << (node & 31);
        node = par[node];
    }
    return bits;
}

// Numerators of a tree tile in fp32, taken apart into operands of 8 (11) significant bits; returns their sum over
// this lane's keys.  Three bf16 operands are a numerator exactly.  Two half operands are it to 2^-24 while the second
// is not subnormal.  Halves are therefore lifted by 2^15, with no score above the reference exponent: this
// then holds for numerators down to 2^-17, and below the error is 2^-41.  The kernel lifts its sums along (powers
// of two: exact).
// m_run: the reference exponent, -inf while the row has seen no key (all scores are -inf then).
template <bool F16> constexpr int kTreeParts = F16 ? 2 : 3;
template <bool F16> constexpr float kTreeLift = F16 ? 15.f : 0.f;          // as a power of two
template <bool F16> constexpr float kTreeUp = F16 ? 0x1p15f : 1.f;
template <bool F16> constexpr float kTreeDown = F16 ? 0x1p-15f : 1.f;
template <bool F16>
__device__ __forceinline__ float tree_numerators(const floatx16 &s, float c, float m_run,
                                                 uint32_t (&parts)[kTreeParts<F16>][8])
{
    const float mc = (m_run == -INFINITY ? 0.f : m_run * c) - kTreeLift<F16>;
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
        float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c, -mc));
        float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], c, -mc));
        sum += p0 + p1;
#pragma unroll
        for (int k = 0; k < kTreeParts<F16>; ++k) {
            const uint32_t u = pack16<F16>(p0, p1);
            parts[k][e >> 1] = u;
            p0 -= low16<F16>(u);
            p1 -= high16<F16>(u);
        }
    }
    return sum;
}

// Output product of a tree tile with these numerators.  frag: the V fragments, f = 16-key half * MT + column tile.
template <bool F16, int MT, int N>
__device__ __forceinline__ void add_tree_product(floatx16 (&o)[MT], const bf16x8 (&frag)[N],
                                                 const uint32_t (&parts)[kTreeParts<F16>][8])
{
#pragma unroll
    for (int k = 0; k < kTreeParts<F16>; ++k)
#pragma unroll
        for (int f = 0; f < N; ++f) {
            const uint32_t *u = parts[k] + 4 * (f / MT);
            o[f % MT] = mfma32<F16>(frag[f], __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3])), o[f % MT]);
        }
}

// Infinite and NaN values of a node must not reach rows that do not see it, but a matrix product carries
// them there (0 * inf).  drop_not_finite replaces them by zeros in the fragments and says whether there were
// any (wave-uniform); if so, add_not_finite puts those of a visible node into the row at the end.
template <bool F16, int N> __device__ __forceinline__ bool drop_not_finite(bf16x8 (&frag)[N])
{
    typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));
    constexpr uint32_t kMagnitude = 0x7fff7fffu, kInf = F16 ? 0x7c00u : 0x7f80u;
    ushortx2 top = {0, 0};
#pragma unroll
    for (int f = 0; f < N; ++f) {
        const uint4 v = __builtin_bit_cast(uint4, frag[f]);
        top = __builtin_elementwise_max(top, __builtin_bit_cast(ushortx2, v.x & kMagnitude));
        top = __builtin_elementwise_max(top, __builtin_bit_cast(ushortx2, v.y & kMagnitude));
        top = __builtin_elementwise_max(top, __builtin_bit_cast(ushortx2, v.z & kMagnitude));
        top = __builtin_elementwise_max(top, __builtin_bit_cast(ushortx2, v.w & kMagnitude));
    }
    if (!__any(top.x >= kInf || top.y >= kInf)) return false;
    auto drop = [](uint32_t x) __attribute__((always_inline)) {
        return ((x & 0x7fffu) >= kInf ? 0u : x & 0xffffu) | ((x >> 16 & 0x7fffu) >= kInf ? 0u : x & 0xffff0000u);
    };
#pragma unroll
    for (int f = 0; f < N; ++f) {
        const uint4 v = __builtin_bit_cast(uint4, frag[f]);
        frag[f] = __builtin_bit_cast(bf16x8, make_uint4(drop(v.x), drop(v.y), drop(v.z), drop(v.w)));
        __builtin_amdgcn_sched_barrier(0);  // few temporaries: the kernels have no registers to spare
    }
    return true;
}

// v_row: the node's value row in global memory; o: the output columns of a lane in half-wave lh.
template <bool F16, int MT>
__device__ __forceinline__ void add_not_finite(floatx16 (&o)[MT], const uint8_t *v_row, int lh)
{
    constexpr uint32_t kInf = F16 ? 0x7c00u : 0x7f80u;
#pragma unroll
    for (int n = 0; n < 4 * MT; ++n) {  // 16-byte chunk n of the row, this half-wave's four elements
        const uint2 x = *(const uint2 *)(v_row + n * 16 + lh * 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t pair = i < 2 ? x.x : x.y;
            const bool bad = ((i & 1 ? pair >> 16 : pair) & 0x7fffu) >= kInf;
            o[n / 4][4 * (n % 4) + i] += bad ? (i & 1 ? high16<F16>(pair) : low16<F16>(pair)) : 0.f;
        }
    }
}

}  // namespace

}  // namespace ls
