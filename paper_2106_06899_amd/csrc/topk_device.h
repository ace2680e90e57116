// Device helpers shared by the kernel sources: order-preserving keys, bf16 conversion,
// and primitives of one 64-lane wave.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace topk {

typedef __bf16 bf16x8 __attribute__((__vector_size__(16)));
typedef float f32x4 __attribute__((__vector_size__(16)));

// ------------------------------------------------------------------ scalar helpers
__device__ __forceinline__ uint32_t ord_u32(float s) {
  uint32_t b = __float_as_uint(s);
  if ((b << 1) == 0u) b = 0u;  // -0 and +0 are the same score
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ord_to_f32(uint32_t u) {
  uint32_t b = (u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u;
  return __uint_as_float(b);
}
__device__ __forceinline__ uint64_t make_key(float s, uint32_t j) {
  return ((uint64_t)ord_u32(s) << 32) | (uint64_t)(0xFFFFFFFFu - j);
}
__device__ __forceinline__ float key_score(uint64_t key) { return ord_to_f32((uint32_t)(key >> 32)); }
__device__ __forceinline__ uint32_t key_index(uint64_t key) { return 0xFFFFFFFFu - (uint32_t)key; }

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {  // nearest-even, finite inputs
  uint32_t b = __float_as_uint(f);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}
template <typename T> __device__ __forceinline__ float load_elem(const void* p, int64_t e);
template <> __device__ __forceinline__ float load_elem<float>(const void* p, int64_t e) {
  return ((const float*)p)[e];
}
template <> __device__ __forceinline__ float load_elem<uint16_t>(const void* p, int64_t e) {
  return bf16_to_f32(((const uint16_t*)p)[e]);
}
template <typename T> __device__ __forceinline__ void store_elem(void* p, int64_t e, float v);
template <> __device__ __forceinline__ void store_elem<float>(void* p, int64_t e, float v) { ((float*)p)[e] = v; }
template <> __device__ __forceinline__ void store_elem<uint16_t>(void* p, int64_t e, float v) {
  ((uint16_t*)p)[e] = f32_to_bf16(v);
}

__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {  // nearest-even, x in the low half
  typedef __bf16 bf16x2 __attribute__((__vector_size__(4)));
  const bf16x2 v = {(__bf16)x, (__bf16)y};
  return __builtin_bit_cast(uint32_t, v);
}

// Eight floats as the exact sums of three bf16 numbers each: the leading 8 significant bits,
// the next 8 and the last 8 (cut off, not rounded, so that nothing is left over). Two values'
// halves are paired up by one byte permute.
__device__ __forceinline__ void split3_bf16(const f32x4& x0, const f32x4& x1, bf16x8 (&part)[3]) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = x0[e], r[4 + e] = x1[e];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = __builtin_amdgcn_perm(__float_as_uint(r[2 * e + 1]), __float_as_uint(r[2 * e]), 0x07060302u);
    part[p] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    if (p < 2)
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] -= __uint_as_float(__float_as_uint(r[e]) & 0xFFFF0000u);
  }
}

// ------------------------------------------------------------------ wave primitives
// Orders one wave's LDS accesses around this point for the compiler; the hardware
// runs a wave's LDS instructions in order, so a wave sees its own earlier writes
// and atomics without a workgroup barrier.
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// lanes of m below this one
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// The value of lane (lane ^ m), m a power of two known at compile time once the
// caller is unrolled: m = 1, 2 by a DPP quad permutation (no LDS traffic), m = 4..16
// by a bit-mode ds_swizzle (xor within 32 lanes), m = 32 by ds_bpermute.
__device__ __forceinline__ uint32_t xor_lane_u32(uint32_t x, int m) {
  switch (m) {
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false);  // quad [1,0,3,2]
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false);  // quad [2,3,0,1]
    case 4: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x1F | (4 << 10));
    case 8: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x1F | (8 << 10));
    case 16: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x1F | (16 << 10));
    default: return (uint32_t)__shfl_xor((int)x, m, 64);
  }
}
__device__ __forceinline__ uint64_t xor_lane_u64(uint64_t x, int m) {
  return ((uint64_t)xor_lane_u32((uint32_t)(x >> 32), m) << 32) | xor_lane_u32((uint32_t)x, m);
}
// The minimum or maximum of x over a wave whose lanes are all active, as a
// wave-uniform value: two DPP quad permutations and the half-row and row mirrors
// leave every row of 16 lanes holding its row's extreme, and the four rows' values
// are read into scalar registers (no LDS traffic, unlike a shuffle).
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme_u32_full(uint32_t x) {
  auto op = [](uint32_t u, uint32_t v) { return MAX ? max(u, v) : min(u, v); };
  x = op(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false));   // quad [1,0,3,2]
  x = op(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false));   // quad [2,3,0,1]
  x = op(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = op(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x140, 0xF, 0xF, false));  // row_mirror
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
  return op(op(r0, r1), op(r2, r3));
}
// The same of floats (NaN if any is).
template <bool MAX>
__device__ __forceinline__ float wave_extreme_f32_full(float x) {
  auto op = [](float u, float v) { return MAX ? __builtin_elementwise_maximum(u, v) : __builtin_elementwise_minimum(u, v); };
  auto dpp = [](float v, auto ctrl) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, false)); };
  x = op(x, dpp(x, std::integral_constant<int, 0xB1>{}));   // quad [1,0,3,2]
  x = op(x, dpp(x, std::integral_constant<int, 0x4E>{}));   // quad [2,3,0,1]
  x = op(x, dpp(x, std::integral_constant<int, 0x141>{}));  // row_half_mirror
  x = op(x, dpp(x, std::integral_constant<int, 0x140>{}));  // row_mirror
  auto at = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
  return op(op(at(0), at(16)), op(at(32), at(48)));
}
// Inclusive prefix sum over the 64 lanes of a wave whose lanes are all active, by
// DPP: row shifts 1, 2, 4, 8 scan each row of 16 lanes, then the broadcasts of lane
// 15 (into rows 1 and 3) and lane 31 (into rows 2 and 3) carry the row totals.
// Lanes without a source add the `old` operand, 0.
__device__ __forceinline__ uint32_t wave_incl_scan_full(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return x;
}

// Bitonic sort, descending, of 64*E keys held as r[e] = element (e*64 + lane); of the first P (a
// power of two) alone where the rest are not needed.
template <int E, int P = 64 * E>
__device__ __forceinline__ void wave_sort_desc(uint64_t (&r)[E]) {
  const int lane = threadIdx.x & 63;
  // fully unrolled: every shuffle distance is a compile-time constant
#pragma unroll
  for (int size = 2; size <= P; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride >= 64) {  // partners in the same lane, other register
        const int rs = stride / 64;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if ((e & rs) == 0) {
            const int i = e * 64 + lane;
            const bool desc = (i & size) == 0;
            const uint64_t x = r[e], y = r[e + rs];
            if ((x < y) == desc) {
              r[e] = y;
              r[e + rs] = x;
            }
          }
        }
      } else {  // partners in another lane, same register
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int i = e * 64 + lane;
          const uint64_t y = xor_lane_u64(r[e], stride);
          const bool desc = (i & size) == 0;
          const bool lower = (lane & stride) == 0;
          // the lower element of a pair keeps the larger key when descending
          const bool keep_max = lower == desc;
          r[e] = keep_max ? (r[e] > y ? r[e] : y) : (r[e] < y ? r[e] : y);
        }
      }
    }
  }
}

}  // namespace topk
