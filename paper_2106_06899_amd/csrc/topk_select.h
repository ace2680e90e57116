// One wave's exact top-k select over keys in registers, and the rows it works on; shared by
// the kernels that end in it.
#pragma once

#include "topk_device.h"
#include "topk_internal.h"

#include <math.h>

namespace topk {

constexpr int CAND_REGS = 16;  // registers per lane for 1024 candidates

// Pass-local row -> (head, query index); false for padding rows of a partial chunk.
struct RowRef {
  int64_t bh, i;
  bool ok;
};
__device__ __forceinline__ RowRef row_of(const Problem& pb, const Pass& ps, int64_t p) {
  int64_t chunk_local, r, id, c;
  RowRef rr;
  if (((uint64_t)p | (uint64_t)pb.C | (uint64_t)(ps.c0 + ps.nc) | (uint64_t)ps.nchunk) >> 31 == 0) {
    // the common case: 32-bit divisions (a few instructions instead of a 64-bit routine)
    const uint32_t cl32 = (uint32_t)p / (uint32_t)pb.C, id32 = (uint32_t)ps.c0 + cl32;
    chunk_local = cl32;
    r = (uint32_t)p - cl32 * (uint32_t)pb.C;
    id = id32;
    rr.bh = id32 / (uint32_t)ps.nchunk;
    c = id32 - (uint32_t)rr.bh * (uint32_t)ps.nchunk;
  } else {
    chunk_local = p / pb.C;
    r = p - chunk_local * pb.C;
    id = ps.c0 + chunk_local;
    rr.bh = id / ps.nchunk;
    c = id - rr.bh * ps.nchunk;
  }
  rr.i = pb.q0 + c * pb.C + r;
  rr.ok = chunk_local < ps.nc && rr.i < pb.q1;
  return rr;
}
__device__ __forceinline__ int64_t valid_keys(const Problem& pb, int64_t i) {
  return pb.causal ? (i + 1 < pb.Lk ? i + 1 : pb.Lk) : pb.Lk;
}

// A candidate word, (raw score bits << 32) | (0xFFFFFFFF - index), as its order key.
__device__ __forceinline__ uint64_t raw_to_key(uint64_t w) {
  return ((uint64_t)ord_u32(__uint_as_float((uint32_t)(w >> 32))) << 32) | (w & 0xFFFFFFFFull);
}

template <int E>
__device__ __forceinline__ void wave_sort_store(const uint64_t* sbuf, uint32_t k_eff, int64_t k, uint64_t* out) {
  const int lane = threadIdx.x & 63;
  uint64_t r[E];
#pragma unroll
  for (int e = 0; e < E; ++e) r[e] = (uint32_t)(e * 64 + lane) < k_eff ? sbuf[e * 64 + lane] : 0ull;
  wave_sort_desc<E>(r);
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * 64 + lane < k) out[e * 64 + lane] = r[e];
}

// Radix select on n <= E * 64 distinct keys held in registers (key[e] is element
// e*64 + lane; elements >= n are ignored). Returns (shift, prefix): the k_eff
// largest keys are exactly those with (key >> shift) >= (prefix >> shift). One
// wave runs it (hist: 256 words of LDS of its own); it synchronises only itself.
// With max_passes, the select stops after that many digits: the set then holds the
// k_eff largest keys and possibly more (the rest of the last digit's bucket), which
// is all a threshold needs.
template <int E>
__device__ __forceinline__ void wave_radix_select(const uint64_t (&key)[E], int n, uint32_t k_eff, uint32_t* hist,
                                                  int* shift_out, uint64_t* prefix_out, int max_passes = 8) {
  const int lane = threadIdx.x & 63;
  uint64_t kmin = ~0ull, kmax = 0ull;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (lane + 64 * e < n) {
      kmin = key[e] < kmin ? key[e] : kmin;
      kmax = key[e] > kmax ? key[e] : kmax;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t a0 = xor_lane_u64(kmin, off), a1 = xor_lane_u64(kmax, off);
    kmin = a0 < kmin ? a0 : kmin;
    kmax = a1 > kmax ? a1 : kmax;
  }
  // bits above the highest differing bit are common to every candidate; the first
  // digit starts at that bit (not at a byte boundary), so it splits the candidates
  // over as many bins as 8 bits can (scores above a threshold often share their top
  // byte, which would pile a byte-aligned first pass onto a few bins)
  const uint64_t diff = kmin ^ kmax;
  int shift = diff == 0 ? 1 : 64 - __builtin_clzll(diff);  // bits [0, shift) differ
  uint64_t prefix = (shift >= 64) ? 0 : (kmax >> shift) << shift;
  uint32_t kr = k_eff;
  for (int pass = 0; pass < max_passes && shift > 0 && kr < (uint32_t)n; ++pass) {
    const int top = shift;  // keys still in play share every bit at or above top
    const int width = top < 8 ? top : 8;
    shift = top - width;
    reinterpret_cast<uint4*>(hist)[lane] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync_lds();
    const uint64_t pre_hi = top >= 64 ? 0 : prefix >> top;
    const uint32_t dmask = (1u << width) - 1u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool match = lane + 64 * e < n && (top >= 64 || (key[e] >> top) == pre_hi);
      if (match) atomicAdd(&hist[(uint32_t)(key[e] >> shift) & dmask], 1u);
    }
    wave_sync_lds();
    const uint4 h4 = reinterpret_cast<const uint4*>(hist)[63 - lane];  // bins 255-4l .. 252-4l
    const uint32_t c4[4] = {h4.w, h4.z, h4.y, h4.x};                   // descending digit order
    const uint32_t local = c4[0] + c4[1] + c4[2] + c4[3];
    uint32_t run = wave_incl_scan_full(local) - local;
    uint32_t digit = 0, above = 0, cnt = 0;
    bool here = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (!here && run < kr && kr <= run + c4[e]) {
        here = true;
        digit = 255u - (uint32_t)(lane * 4 + e);
        above = run;
        cnt = c4[e];
      }
      run += c4[e];
    }
    const uint64_t who = __ballot(here);
    const int src = __builtin_ctzll(who);  // wave-uniform
    digit = (uint32_t)__builtin_amdgcn_readlane((int)digit, src);
    above = (uint32_t)__builtin_amdgcn_readlane((int)above, src);
    cnt = (uint32_t)__builtin_amdgcn_readlane((int)cnt, src);
    wave_sync_lds();  // hist is cleared again by the next pass
    prefix |= (uint64_t)digit << shift;
    kr -= above;
    if (cnt == kr) break;  // every key of this bucket is selected
  }
  *shift_out = shift;
  *prefix_out = prefix;
}

// The k_eff <= 64 * E distinct keys of sbuf, stored in descending order (the first
// 64 * E of k words, 0 pads): each key goes to its rank, the number of larger keys,
// counted against every key through broadcast LDS reads. Two VALU per comparison:
// at E = 1 faster than the bitonic network (measured slower at E = 2).
template <int E>
__device__ __forceinline__ void wave_rank_store(const uint64_t* sbuf, uint32_t k_eff, int64_t k, uint64_t* out) {
  const int lane = threadIdx.x & 63;
  uint64_t x[E];
  uint32_t rank[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    x[e] = (uint32_t)(e * 64 + lane) < k_eff ? sbuf[e * 64 + lane] : 0ull;
    rank[e] = 0;
  }
#pragma unroll 8
  for (uint32_t j = 0; j < k_eff; ++j) {
    const uint64_t y = sbuf[j];
#pragma unroll
    for (int e = 0; e < E; ++e) rank[e] += y > x[e] ? 1u : 0u;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * 64 + lane;
    if ((uint32_t)t < k_eff) out[rank[e]] = x[e];
    else if (t < k) out[t] = 0ull;
  }
}

// The k_eff (<= KCAP: 256 or 512) largest of n <= E * 64 register keys, sorted
// descending, written as k words to out (0 pads). sbuf: KCAP keys of LDS.
template <int E, int KCAP = 256>
__device__ __forceinline__ void wave_select_store(const uint64_t (&key)[E], int n, uint32_t k_eff, int64_t k,
                                                  uint64_t* sbuf, uint32_t* hist, uint64_t* out) {
  const int lane = threadIdx.x & 63;
  int shift;
  uint64_t prefix;
  wave_radix_select<E>(key, n, k_eff, hist, &shift, &prefix);
  // selected: (key >> shift) >= (prefix >> shift); compact them into sbuf
  const uint64_t lim = prefix >> shift;
  int base = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool take = lane + 64 * e < n && (key[e] >> shift) >= lim;
    const uint64_t m = __ballot(take);
    const int pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (take && pos < KCAP) sbuf[pos] = key[e];
    base += __popcll(m);
  }
  wave_sync_lds();
  int sorted;
  if (k_eff <= 64) wave_rank_store<1>(sbuf, k_eff, k, out), sorted = 64;
  else if (k_eff <= 128) wave_sort_store<2>(sbuf, k_eff, k, out), sorted = 128;
  else if (KCAP <= 256 || k_eff <= 256) wave_sort_store<4>(sbuf, k_eff, k, out), sorted = 256;
  else wave_sort_store<(KCAP > 256 ? 8 : 4)>(sbuf, k_eff, k, out), sorted = 512;
  for (int64_t t = lane + sorted; t < k; t += 64) out[t] = 0ull;
}

// ------------------------------------------------------------------ team primitives
// A "team" is one workgroup of NT threads (NT = 64 or 256); all sync is __syncthreads.
template <int NT>
__device__ __forceinline__ uint32_t team_excl_scan(uint32_t x, uint32_t* tmp) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t incl = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (NT == 64) return incl - x;
  if (lane == 63) tmp[w] = incl;
  __syncthreads();
  uint32_t base = 0;
  for (int q = 0; q < w; ++q) base += tmp[q];
  __syncthreads();
  return base + incl - x;
}

// Digits a sampled threshold resolves: the sign, the exponent and the top 7 bits of the
// mantissa of the R-th largest sample (finer resolution only trims a few candidates).
constexpr int THRESH_PASSES = 2;

// Exact radix select of the k_eff largest keys among n (distinct) 64-bit keys,
// 8 bits per pass from the top. On return the selected set is exactly
// { key : (key >> shift) >= (prefix >> shift) }. With max_passes < 8 it stops early
// and the set holds the k_eff largest keys and possibly more (the rest of the last
// digit's bucket), which is all a threshold needs.
template <int NT, class GetKey>
__device__ void team_radix_select(const GetKey& getkey, int64_t n, uint32_t k_eff, uint32_t* hist,
                                  uint32_t* misc, int* shift_out, uint64_t* prefix_out, int max_passes = 8) {
  uint64_t prefix = 0;
  int shift = 64;
  uint32_t kr = k_eff;
  for (int pass = 0; pass < max_passes; ++pass) {
    shift -= 8;
    for (int b = threadIdx.x; b < 256; b += NT) hist[b] = 0;
    __syncthreads();
    for (int64_t e = threadIdx.x; e < n; e += NT) {
      const uint64_t key = getkey(e);
      const bool match = pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8));
      if (match) atomicAdd(&hist[(uint32_t)(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    constexpr int BPT = 256 / NT;
    uint32_t c[BPT];
    uint32_t local = 0;
#pragma unroll
    for (int e = 0; e < BPT; ++e) {
      c[e] = hist[255 - (threadIdx.x * BPT + e)];  // bins in descending digit order
      local += c[e];
    }
    uint32_t run = team_excl_scan<NT>(local, misc);
#pragma unroll
    for (int e = 0; e < BPT; ++e) {
      if (run < kr && kr <= run + c[e]) {
        misc[4] = 255u - (uint32_t)(threadIdx.x * BPT + e);
        misc[5] = run;
        misc[6] = c[e];
      }
      run += c[e];
    }
    __syncthreads();
    const uint32_t digit = misc[4], above = misc[5], cnt = misc[6];
    __syncthreads();
    prefix |= (uint64_t)digit << shift;
    kr -= above;
    if (cnt == kr) break;  // every key of this bucket is selected
  }
  *shift_out = shift;
  *prefix_out = prefix;
}

// Bitonic sort of P (power of two) keys in LDS, descending.
template <int NT>
__device__ void team_sort_desc(uint64_t* s, int P) {
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = threadIdx.x; t < (P >> 1); t += NT) {
        const int i = 2 * stride * (t / stride) + (t % stride);
        const int j = i + stride;
        const bool desc = (i & size) == 0;
        const uint64_t a = s[i], b = s[j];
        if ((a < b) == desc) {
          s[i] = b;
          s[j] = a;
        }
      }
      __syncthreads();
    }
  }
}

// Select the k_eff largest of n keys, sort them and write k words to out (0 pads).
// sbuf holds P >= k_eff keys (power of two).
template <int NT, class GetKey>
__device__ void team_topk(const GetKey& getkey, int64_t n, uint32_t k_eff, uint32_t k, uint64_t* sbuf, int P,
                          uint32_t* hist, uint32_t* misc, uint64_t* out) {
  int shift;
  uint64_t prefix;
  team_radix_select<NT>(getkey, n, k_eff, hist, misc, &shift, &prefix);
  const uint64_t lim = prefix >> shift;
  if (threadIdx.x == 0) misc[7] = 0;
  for (int t = threadIdx.x; t < P; t += NT) sbuf[t] = 0;
  __syncthreads();
  for (int64_t e = threadIdx.x; e < n; e += NT) {
    const uint64_t key = getkey(e);
    if ((key >> shift) >= lim) {
      const uint32_t pos = atomicAdd(&misc[7], 1u);
      if (pos < (uint32_t)P) sbuf[pos] = key;
    }
  }
  __syncthreads();
  team_sort_desc<NT>(sbuf, P);
  for (uint32_t t = threadIdx.x; t < k; t += NT) out[t] = t < k_eff ? sbuf[t] : 0ull;
}

__host__ __device__ __forceinline__ int pow2_at_least(int64_t x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

// Writes a row's selection from sorted keys (k words, 0 pads) as the debug outputs: indices
// and raw scores, padded with -1 and -inf. One wave; key: word t of the row.
template <class GetKey>
__device__ __forceinline__ void write_selection(const Problem& pb, int64_t grow, uint32_t k_eff, int lane0, int lanes,
                                                const GetKey& key) {
  for (int64_t t = lane0; t < pb.k; t += lanes) {
    const uint64_t w = t < k_eff ? key(t) : 0ull;
    if (pb.idx_out) pb.idx_out[grow * pb.k + t] = t < k_eff ? (int32_t)key_index(w) : -1;
    if (pb.score_out) pb.score_out[grow * pb.k + t] = t < k_eff ? key_score(w) : -INFINITY;
  }
}

}  // namespace topk
