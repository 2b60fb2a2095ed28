// Device-side helpers shared by the HIP kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "divmagic.h"

namespace sc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// the same for addresses that are only element-aligned (the hardware takes them)
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Round to nearest even (the gfx950 conversion instruction rounds RNE).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  __bf16 h = static_cast<__bf16>(f);
  return __builtin_bit_cast(uint16_t, h);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
}

// n / d for n < 2^31 with a host-computed magic pair (divmagic.h).
__device__ __forceinline__ uint32_t fast_div(uint32_t n, DivMagic m) {
  return (__umulhi(n, m.mul) + n) >> m.shift;
}

// Work-group index remap for the 8 XCDs of MI355X: consecutive hardware
// work-group ids are dealt round-robin to the XCDs, so hand each XCD a
// contiguous range of logical work items (which then share its L2).
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t n) {
  const uint32_t x = b & 7u, local = b >> 3, per = n >> 3, extra = n & 7u;
  return x * per + (x < extra ? x : extra) + local;
}

// N <= 4 copies of 1 KB each from memory straight into consecutive LDS: lane i
// of copy j moves 16 bytes from biased + off[j] + 1024 j to lds + 1024 j + 16 i.
// The instruction's offset field moves the memory and the LDS address alike, so
// M0, which carries the LDS address, is set once for the group (and restored);
// off[j] makes up for it (kCopyBias - 1024 j above the lane's own offset, the base kCopyBias
// lower, so that it stays non-negative; the callers see to it
// that it stays below 2^32).  Written as inline asm: while a copy
// it knows of is in flight, the compiler waits for every LDS fragment read with
// lgkmcnt(0); not knowing of these, it counts the reads exactly.  The copies
// complete under the caller's explicit vmcnt waits.
constexpr uint32_t kCopyBias = 3072;
template <int N>
__device__ __forceinline__ void copy_group(const char* biased, const uint32_t* off, uint32_t lds) {
  uint32_t saved;
  static_assert(N >= 1 && N <= 4, "copies per group");
  if constexpr (N == 1)
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %3, %1\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(biased), "s"(lds), "v"(off[0])
        : "memory");
  else if constexpr (N == 2)
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %3, %1\n\t"
        "global_load_lds_dwordx4 %4, %1 offset:1024\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(biased), "s"(lds), "v"(off[0]), "v"(off[1])
        : "memory");
  else if constexpr (N == 3)
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %3, %1\n\t"
        "global_load_lds_dwordx4 %4, %1 offset:1024\n\t"
        "global_load_lds_dwordx4 %5, %1 offset:2048\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(biased), "s"(lds), "v"(off[0]), "v"(off[1]), "v"(off[2])
        : "memory");
  else
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %3, %1\n\t"
        "global_load_lds_dwordx4 %4, %1 offset:1024\n\t"
        "global_load_lds_dwordx4 %5, %1 offset:2048\n\t"
        "global_load_lds_dwordx4 %6, %1 offset:3072\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(biased), "s"(lds), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3])
        : "memory");
}

}  // namespace sc
