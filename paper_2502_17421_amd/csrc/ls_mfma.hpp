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

}  // namespace

}  // namespace ls
