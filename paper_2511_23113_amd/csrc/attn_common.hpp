// Device helpers the attention kernels share: vector types, bf16 packing, lane-pair exchange,
// direct global -> LDS copies.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The speculative softmax redoes a unit when a lane's sum of its 16 probabilities exceeds this:
// then some score is above the running max by about six powers of two or more (16 probabilities
// at or below 1 sum to less than the limit; until it trips, P may exceed 1 by at most this
// factor, which f32 / bf16 hold without loss).
constexpr float SPEC_SUM_LIMIT = 64.0f;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  f32x2 f = {a, b};
  bf16x2 h = __builtin_convertvector(f, bf16x2);  // round-to-nearest-even
  return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 u) { return __builtin_bit_cast(bf16x8, u); }

// Exchange between the lane pair (r, r + 32) with one VALU swap of the two 32-lane halves (no
// LDS traffic): v_permlane32_swap swaps the upper half of its first operand with the lower half
// of its second; fed two copies of x it leaves {lo, lo} in the first and {hi, hi} in the second.
// Inline assembly: the compiler's builtin returns the first register for both results.  The
// s_nop's cover the wait states between a VALU write and the swap's read of the same register,
// and between the swap and its consumers, which the compiler cannot insert inside an asm block.
struct halves { float lo, hi; };
__device__ __forceinline__ halves swap_halves(float x) {
  float a = x, b = x;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return {a, b};
}
__device__ __forceinline__ float max_xor32(float x) {
  const halves sw = swap_halves(x);
  return fmaxf(sw.lo, sw.hi);
}
__device__ __forceinline__ float sum_xor32(float x) {
  const halves sw = swap_halves(x);
  return sw.lo + sw.hi;
}

// The swap itself: the upper half (lanes 32..63) of a and the lower half of b change places.
__device__ __forceinline__ void swap_upper_lower(uint32_t& a, uint32_t& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}

// Direct global -> LDS copies.  One global_load_lds_dwordx4 moves 64 x 16 bytes: lane i reads
// 16 bytes at base + voff(i) + OFF and they land at LDS byte address M0 + OFF + 16*i; the
// instruction offset applies to both sides, so the copies of one group share a base and an M0.
// Inline assembly keeps the copies outside the compiler's wait-count bookkeeping: the kernel waits for them itself, by
// count.  What a wait or a barrier publishes has to be older than the N youngest of the wave's vector memory operations
// at its s_waitcnt vmcnt(N): where two query groups share their slices, N is at most 4 x LOADS in front of a slice's
// barrier, the copies of the last two slices, so every slice has to issue its 2 x LOADS copies, also past the end of the list
// (other operations among them only make it wait for more).  Between set_copy_dst and the last copy of its group M0 must not
// change.  A group goes on over other sub-slots, the end of a step and the redone softmax behind it, and the asm
// says nothing of M0: the kernels use nothing else that sets it, which a test reads from their listing.
// No "memory" clobber: LDS reads of the OTHER buffer may be scheduled across a copy.
__device__ __forceinline__ void set_copy_dst(uint32_t lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(lds_dst));
}
template <int OFF>
__device__ __forceinline__ void copy16_to_lds(const unsigned char* base, uint32_t voff) {
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(voff), "s"(base), "n"(OFF));
}
// copy number n (0..3) of a group: byte offset n KiB
__device__ __forceinline__ void copy16_nth(int n, const unsigned char* base, uint32_t voff) {
  if (n == 0) copy16_to_lds<0>(base, voff);
  else if (n == 1) copy16_to_lds<1024>(base, voff);
  else if (n == 2) copy16_to_lds<2048>(base, voff);
  else copy16_to_lds<3072>(base, voff);
}

}  // namespace
