// Device helpers shared by the gfx950 decode kernels (bf16 cache and fp8 cache).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.h"

namespace omniattn {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

#define LDS_PTR(T, byte_off) ((__attribute__((address_space(3))) T*)(uintptr_t)(byte_off))

__device__ __forceinline__ bool retained(int j, int L, int S, int W) {
  return j < L && (j < S || j >= L - W);
}

// Direct global->LDS load of 16 bytes per lane: lane l's bytes land at LDS address
// M0 + IMM + 16 l and are read from base + off + IMM (base wave-uniform, off per lane;
// the instruction's immediate offset applies to both sides).  Written as assembly so
// that the compiler does not treat it as a store that may alias every later LDS read
// and drain the whole prefetch before the first read of another stage; completion is
// awaited explicitly (wait_vm) before the barrier that publishes the tile.
// M0 carries the LDS base.  Nothing else in these kernels uses M0 (no indirect register
// addressing, no GWS, no compiler-issued LDS-DMA), so it is simply overwritten.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma_set_lds_base(uint32_t lds_base) {
  const uint32_t slds = __builtin_amdgcn_readfirstlane(lds_base);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(slds) : "m0");
}
template <int IMM>
__device__ __forceinline__ void dma16(const uint8_t* base, uint32_t off) {
  // wave-uniform by construction; make that visible to the register allocator
  const uint64_t b = (uint64_t)(uintptr_t)base;
  const uint32_t b_lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
  const uint32_t b_hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  const uint64_t sbase = ((uint64_t)b_hi << 32) | b_lo;
  // nt: cache rows are read once per work unit; marking them as streaming keeps them from
  // pushing Q (shared by the units of a sequence) and the partial results out of the caches
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2 nt" : : "v"(off), "s"(sbase), "n"(IMM) : "m0");
}
#pragma clang diagnostic pop
// Wait until at most N of this wave's vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Direct global->LDS loads (see dma16 for what they do), each with its LDS base.  Base and LDS address
// come fresh from vector registers (v_readfirstlane), and the compiler does not see the memory
// instruction inside the assembly: the five wait states that a vector-memory instruction needs behind
// such a write of its scalar address stand in the same block.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ uint64_t uniform64(uint64_t b) {
  return ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
}
template <bool NT>  // nt: rows read once per work unit (see dma16), also where several head blocks read them
__device__ __forceinline__ void load_lds16(uint32_t lds, const uint8_t* base, uint32_t off) {
  const uint64_t b = uniform64((uint64_t)(uintptr_t)base);
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds);
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2 nt" : : "s"(m), "v"(off), "s"(b) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(m), "v"(off), "s"(b) : "m0", "memory");
}
__device__ __forceinline__ void load_lds4(uint32_t lds, const uint8_t* base, uint32_t off) {
  const uint64_t b = uniform64((uint64_t)(uintptr_t)base);
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2" : : "s"(m), "v"(off), "s"(b) : "m0", "memory");
}
// The same at the LDS base set before, from scalar addresses that went through settle_address.
// load_lds4_at: for the lanes of a mask (all lanes of the wave must be active).
__device__ __forceinline__ void set_lds_base(uint32_t lds) {
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(m) : "m0");
}
__device__ __forceinline__ void settle_address(uint64_t& a, uint64_t& b) {
  a = uniform64(a);
  b = uniform64(b);
  asm volatile("s_nop 4" : "+s"(a), "+s"(b));
}
template <int IMM>
__device__ __forceinline__ void load_lds16_at(uint64_t base, uint32_t off) {
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2 nt" : : "v"(off), "s"(base), "n"(IMM) : "m0", "memory");
}
__device__ __forceinline__ void load_lds4_at(uint64_t lanes, uint64_t base, uint32_t off) {
  asm volatile("s_mov_b64 exec, %0\n\tglobal_load_lds_dword %1, %2\n\ts_mov_b64 exec, -1" : : "s"(lanes), "v"(off), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop

// Exchange of rows of 16 lanes (halves of 32) between two registers: with a = b = x before, a and b hold the
// lane's own value and that of lane ^ 16 (lane ^ 32) behind it, in an order that depends on the lane.
// (Assembly: with the builtin the compiler drops one of two results that are combined at once.  The wait
// states are the ones it places for the builtin.)
__device__ __forceinline__ void swap16(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}

// Four bf16 query elements (two words) in two e4m3 terms, q = 2^ex (hi + lo / 16): .x the high terms, .y the low ones.
// scale = 2^ex, inv = 2^-ex, both normal.  Seven instructions for two elements: the scaled conversion takes the bf16 pair
// as it is, and the remainder is one fused multiply-add (the product with a power of two is exact).  An element that is NaN or
// an infinity leaves a NaN code in its terms (the conversions do not saturate), and the row's result is NaN.
constexpr int kQLoShift = 4;  // the low term is stored 16 times too large
__device__ __forceinline__ u32x2 split_q4(uint32_t w0, uint32_t w1, float scale, float inv) {
  typedef __attribute__((ext_vector_type(2))) short s16x2;
  s16x2 hi = {0, 0}, lo = {0, 0};
  auto two = [&](uint32_t w, auto upper_tag) {
    constexpr bool upper = decltype(upper_tag)::value;
    hi = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(hi, __builtin_bit_cast(bf16x2, w), scale, upper);
    const f32x2 back = __builtin_amdgcn_cvt_pk_f32_fp8(__builtin_bit_cast(int, hi), upper);
    lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(lo, fmaf(__builtin_bit_cast(float, w << 16), inv, -back[0]),
                                                  fmaf(__builtin_bit_cast(float, w & 0xffff0000u), inv, -back[1]), 1.0f / (1 << kQLoShift), upper);
  };
  two(w0, std::false_type{});
  two(w1, std::true_type{});
  return u32x2{__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo)};
}
// The larger of mx and the magnitudes of four bf16 numbers (two words), in the upper half of a float: a word as a float is its
// upper number, the lower ones are needed shifted up in any case.  NaN is passed over, and so is an infinity whose word reads
// as NaN (see above for what becomes of such a row).
__device__ __forceinline__ float bf16_max4(float mx, uint32_t w0, uint32_t w1) {
  mx = fmaxf(fmaxf(mx, fabsf(__builtin_bit_cast(float, w0))), fabsf(__builtin_bit_cast(float, w1)));
  return fmaxf(fmaxf(mx, fabsf(__builtin_bit_cast(float, w0 << 16))), fabsf(__builtin_bit_cast(float, w1 << 16)));
}
// The exponent for a row whose largest magnitude has the bits m: that goes to [128, 256), as far as scale and inv are normal.
// (A row of subnormal numbers, multiples of 2^-133 below 2^-126, becomes multiples of 2^-7 below 1: exact in the two terms.)
__device__ __forceinline__ int split_q_exponent(int m) {
  const int e = m >> 7;
  const int ex = (e > 254 ? 254 : e) - 127 - 7;
  return ex < -126 ? -126 : ex;
}
// What the row's raw products are multiplied by.  Never 0: a masked position's -infinity has to survive it.  (Subnormal, it is
// off by at most 2^-150, a logit by 2^-22.)
__device__ __forceinline__ float split_q_factor(float scale_log2, int ex) {
  return fmaxf(__builtin_amdgcn_ldexpf(fabsf(scale_log2), ex), 0x1p-149f);
}

// The XCD (accelerator complex die) this wave runs on: compute units of one XCD share an L2.
__device__ __forceinline__ uint32_t xcc_id() {
  uint32_t id;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
  return id & 15u;
}

}  // namespace omniattn
