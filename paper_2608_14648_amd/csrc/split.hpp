// fp32 products on the fp16 matrix cores.
//
// A value v scaled by a power of two s is written as hi + lo with hi = fp16(s v) and
// lo = fp16(s v - hi), both to nearest even: hi keeps 11 significant bits and lo the
// next 11, so hi + lo is s v to within max(2^-23 |s v|, 2^-25), the second term being
// half of fp16's subnormal spacing.  A dot product becomes hi hi' + hi lo' + lo hi'
// with fp32 accumulation (lo lo' is below 2^-22 of the product): three
// v_mfma_f32_32x32x16_f16 of 32 cycles do the work of eight v_mfma_f32_32x32x2_f32 of
// 64.
//
// The instruction adds 8 products at a time to the accumulator (probed on the
// device), so a dot product is rounded six times per 16 dims where the fp32
// instruction rounds 16 times, which outweighs what the split leaves out: scores end
// up closer to 64-bit sums than the fp32 kernel's (relative error of the winning
// score, fp32 kernel -> split: 3.8e-7 -> 2.5e-7 at d = 64, 4.5e-7 -> 2.7e-7 at 256,
// 8.3e-7 -> 5.1e-7 at 768).  But each addition also cuts a few bits below the
// accumulator towards zero, 2^-10 of an ulp on average: the mean of many scores is off
// by 2e-11 d, under half an ulp of one score, and sums over points of the small
// difference ||x||^2 + score must not be made of them (the objective is summed from
// the distances themselves, direct_objective_kernel).
#pragma once

#include "common.hpp"

namespace kmq {

typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));

// Two floats scaled by s and split: the packed hi and lo pairs.  Four v_fma_mix (the
// scaling is part of the conversion).
__device__ __forceinline__ void split2(float v0, float v1, float s, uint32_t &hi, uint32_t &lo) {
  const h16x2 h = {(_Float16)__builtin_fmaf(v0, s, 0.0f), (_Float16)__builtin_fmaf(v1, s, 0.0f)};
  hi = __builtin_bit_cast(uint32_t, h);
  // hide how the pair was made, so that the residuals read its halves in place
  // (op_sel) instead of converting each value a second time
  asm("" : "+v"(hi));
  const h16x2 hp = __builtin_bit_cast(h16x2, hi);
  const h16x2 l = {(_Float16)__builtin_fmaf(v0, s, -(float)hp[0]), (_Float16)__builtin_fmaf(v1, s, -(float)hp[1])};
  lo = __builtin_bit_cast(uint32_t, l);
}

// Direct copy of 16 bytes per lane (4 bytes in lds_copy4) from a wave-uniform base
// plus a per-lane byte offset into LDS: the wave's 64 lanes fill 1 KB (256 bytes) at
// LDS byte address lds (wave-uniform) in lane order.  The caller waits (vmcnt)
// before the barrier that publishes the data.
typedef __attribute__((address_space(3))) uint8_t lds_byte;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_copy16_at(const void *base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
__device__ __forceinline__ void lds_copy4_at(const void *base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// (score, index) keys as in the other assignment kernels: the order of the keys is
// the order of (score, index), -0 taken as +0
__device__ __forceinline__ unsigned long long split_key(float sc, int idx) {
  uint32_t u = __float_as_uint(sc == 0.0f ? 0.0f : sc);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << 32) | (uint32_t)idx;
}

}  // namespace kmq
