// Short rows in one kernel: top-k attention (Eq. 4) and the feed-forward recast (Eq. 3)
// where every score of a row fits a workgroup's LDS (at most 1024 keys). One launch takes
// the place of the score, select, fallback and finalize launches, and nothing but the
// output leaves the chip.
//
// A workgroup owns TR = 16 or 32 consecutive query rows of one head; its E waves (64 E
// threads) each own 64 of the row's 64 E key slots:
//  1. scores: each wave multiplies its keys with the TR queries by 16x16 matrix
//     instructions (bf16: 16x16x32; fp32: 16x16x4, exact 32-bit products and sums) and
//     writes them to LDS. Operands are read straight from global memory in 16-byte parts:
//     the contraction is free to take the features in any order, so lane group g takes
//     features g * FB .. + FB - 1 of every group of 4 FB (FB elements per 16 bytes);
//  2. select: each wave takes TR / E rows, one at a time, E scores per lane in registers.
//     The k-th largest score is found by counting (ballots) the scores at or above a
//     threshold that interpolates between bounds holding more and fewer than k, on the
//     scores' order-preserving keys; a threshold that leaves exactly k ends the search
//     (about 7 steps on Gaussian scores), ties at the k-th score are broken by index. The
//     row's weights (0 where not selected) replace its scores in LDS;
//  3. values: out = P V by the matrix instructions, P in full 32 bits: fp32 values by the
//     fp32 instruction, bf16 values with every weight taken apart into three bf16 numbers
//     that add up to it exactly (the products and sums are 32-bit; with two numbers, 16 or
//     17 bits, 96 heads of 512 took 67 us for 69, but 2.2e-3 of the stored values were not
//     the 64-bit result rounded, against 1.7e-4). Each wave takes
//     its 64 keys, a value row is read as one contiguous part per lane (column n * CPL + c
//     is column n of tile c), and the waves' partial sums are added in a fixed order.
// A dense P V reads each value row once per TR query rows: at 512 keys and k = 64 that is
// 2 KB a row instead of the 8 KB that a gather of the selected rows moves.
//
// Bound by the select's vector instructions (about 350 per row at 512 keys, half of the
// kernel's time) and by latency. Against the launches it replaced (every score written as
// an 8-byte candidate, selected from global memory, value rows gathered): 96 heads of 512
// tokens, d = 64, bf16, k = 64: 240 -> 69 us; 48 heads of 1024: 580 -> 184 us with the
// cache outputs; one fp32 head of 1024, k = 32 (64 workgroups, latency): 31 -> 25 us of
// kernel time in one launch instead of five.
//
// A result that is not finite (an infinite or NaN value row that a zero weight met) is
// computed again, for its row only, by a sum over the selected keys alone.
#include "topk_device.h"
#include "topk_internal.h"

#include <math.h>

#include <type_traits>

namespace topk {

struct RowsArgs {
  const void* Q;
  const void* K;
  const void* V;
  void* out;
  int64_t Lq, tiles_per_head, kv_head_stride;
  int64_t first;        // first workgroup of this launch
  int Lk, k, causal, act;
  float c;              // softmax: scale * log2(e)
  int32_t* idx_out;
  float* score_out;
  int scratch;          // 64-bit words of sort scratch per wave (a power of two >= k), 0 without outputs
};

__device__ __forceinline__ f32x4 mfma_step(uint4 a, uint4 b, f32x4 acc, uint16_t) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_step(uint4 a, uint4 b, f32x4 acc, float) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}

// The sum of x over a wave whose lanes are all active.
__device__ __forceinline__ float rows_wave_sum(float x) {
  auto dpp = [](float v, auto ctrl) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, false)); };
  x += dpp(x, std::integral_constant<int, 0xB1>{});
  x += dpp(x, std::integral_constant<int, 0x4E>{});
  x += dpp(x, std::integral_constant<int, 0x141>{});
  x += dpp(x, std::integral_constant<int, 0x140>{});
  auto at = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
  return (at(0) + at(16)) + (at(32) + at(48));
}
__device__ __forceinline__ float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }

// Writes a row's n <= P distinct selected keys (in scratch, a wave's own LDS) in
// descending order as indices and raw scores, padded to k <= P with -1 and -inf.
template <int E, int P = 64 * E>
__device__ __forceinline__ void rows_sorted_out(const uint64_t* scratch, int n, int k, int32_t* idx, float* sc) {
  const int lane = threadIdx.x & 63;
  uint64_t r[E];
#pragma unroll
  for (int e = 0; e < E; ++e) r[e] = e * 64 + lane < n ? scratch[e * 64 + lane] : 0ull;
  wave_sort_desc<E, P>(r);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int t = e * 64 + lane;
    if (t < k) {
      if (idx) idx[t] = t < n ? (int32_t)key_index(r[e]) : -1;
      if (sc) sc[t] = t < n ? key_score(r[e]) : -INFINITY;
    }
  }
}

template <typename T, int D, int E, int TR>
__global__ __launch_bounds__(64 * E, 4) void k_rows(RowsArgs a) {
  constexpr int FB = 16 / (int)sizeof(T);  // elements per 16-byte part
  constexpr int NG = D / (4 * FB);         // feature groups (one 16-byte part per lane each)
  constexpr int CG = NG < 4 ? NG : 4;      // groups whose operands are held at once
  constexpr int RT = TR / 16;              // 16-row tiles
  constexpr int LKP = 64 * E;              // key slots
  constexpr int LDS_ROW = LKP + 4;         // row stride of the score tile
  constexpr int CPL = D / 16;              // value columns per lane,
  constexpr int CPP = CPL == 8 ? 4 : CPL;  // read CPP at a time
  constexpr bool F32 = sizeof(T) == 4;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float inv_lds[TR];
  __shared__ int bad_lds[TR];
  float* S = sm;                                            // [TR][LDS_ROW] scores, then weights
  uint64_t* scratch = (uint64_t*)(sm + TR * LDS_ROW);       // [E][a.scratch]
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive row tiles of a head on one XCD (its L2 holds the head's keys and values)
  const int64_t NGR = gridDim.x, bid = blockIdx.x;
  const int64_t wg = a.first + ((NGR % 8 == 0) ? (bid % 8) * (NGR / 8) + bid / 8 : bid);
  const int64_t bh = wg / a.tiles_per_head, i0 = (wg - bh * a.tiles_per_head) * TR;
  const T* Qt = (const T*)a.Q + (bh * a.Lq + i0) * D;
  const T* Kh = (const T*)a.K + bh * a.kv_head_stride;
  const T* Vh = (const T*)a.V + bh * a.kv_head_stride;
  const int64_t last = i0 + TR - 1 < a.Lq - 1 ? i0 + TR - 1 : a.Lq - 1;
  const int nkeys = a.causal && last + 1 < a.Lk ? (int)last + 1 : a.Lk;  // keys any row of the tile may see
  const int key0 = wave * 64;
  const bool live = key0 < nkeys;  // this wave's keys matter to some row

  // second pass (mode 1): only when a result of the first was not finite
  for (int mode = 0; mode < 2; ++mode) {
    // opaque to the compiler, so that it keeps no address of one pass for the other
    int lane = tid & 63;
    asm volatile("" : "+v"(lane));
    const int n = lane & 15, g = lane >> 4;
    if (live) {
      f32x4 acc[4][RT];
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[t][r] = (f32x4){};
#pragma unroll
      for (int c0 = 0; c0 < NG; c0 += CG) {
        if (D > 64) __builtin_amdgcn_sched_barrier(0);
        uint4 qf[RT][CG];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          // rows past the head's end repeat its last row (their results are not stored)
          const uint32_t qo = (uint32_t)min(16 * r + n, (int)(last - i0)) * D + g * FB;
#pragma unroll
          for (int s = 0; s < CG; ++s)
            if (c0 + s < NG) qf[r][s] = *(const uint4*)(Qt + qo + (c0 + s) * 4 * FB);
        }
        constexpr int TB = TR == 16 ? 4 : D == 128 ? 1 : F32 || D > 64 ? 2 : 4;  // key tiles whose operands are in flight together
#pragma unroll
        for (int t0 = 0; t0 < 4; t0 += TB) {
          if (D > 64) __builtin_amdgcn_sched_barrier(0);
          uint4 kf[TB][CG];
#pragma unroll
          for (int t = 0; t < TB; ++t) {
            int j = key0 + 16 * (t0 + t) + n;
            j = j < a.Lk ? j : a.Lk - 1;
#pragma unroll
            for (int s = 0; s < CG; ++s)
              if (c0 + s < NG) kf[t][s] = *(const uint4*)(Kh + (uint32_t)(j * D + g * FB) + (c0 + s) * 4 * FB);
          }
#pragma unroll
          for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int s = 0; s < CG; ++s)
              if (c0 + s < NG)
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[t0 + t][r] = mfma_step(kf[t][s], qf[r][s], acc[t0 + t][r], T());
        }
      }
      // lane: query n of row tile r, keys 4 g .. 4 g + 3 of key tile t
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < RT; ++r)
          *(f32x4*)&S[(16 * r + n) * LDS_ROW + key0 + 16 * t + 4 * g] = acc[t][r];
    }
    __syncthreads();

    // ---- select and weights, one row per wave at a time: element e = 4 c + i of a lane is
    // key 256 c + 4 lane + i (16-byte LDS reads)
    for (int r = wave; r < TR; r += E) {
      const int64_t i = i0 + r;
      float* row = S + r * LDS_ROW;
      if (i > last) {
#pragma unroll
        for (int c = 0; c < E / 4; ++c) *(f32x4*)&row[256 * c + 4 * lane] = (f32x4){};
        continue;
      }
      const int nv = a.causal && i + 1 < a.Lk ? (int)i + 1 : a.Lk;
      const int k_eff = a.k < nv ? a.k : nv;
      float s[E], mx = -INFINITY, mn = INFINITY;
#pragma unroll
      for (int c = 0; c < E / 4; ++c) {
        const f32x4 x = *(const f32x4*)&row[256 * c + 4 * lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) s[4 * c + q] = x[q];
      }
      auto key_of = [&](int e) { return 256 * (e >> 2) + 4 * lane + (e & 3); };
      // extremes of the valid scores (the NaN-propagating ones, which need no canonicalising)
      if (nv < LKP) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const bool ok = key_of(e) < nv;
          mn = __builtin_elementwise_minimum(mn, ok ? s[e] : INFINITY);
          s[e] = ok ? s[e] : -INFINITY;
          mx = __builtin_elementwise_maximum(mx, s[e]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          mn = __builtin_elementwise_minimum(mn, s[e]);
          mx = __builtin_elementwise_maximum(mx, s[e]);
        }
      }
      mx = wave_extreme_f32_full<true>(mx);
      mn = wave_extreme_f32_full<false>(mn);
      // bounds of the k-th largest score: at least k are >= lo (clo of them), fewer than k
      // are >= hi (chi of them)
      float lo = mn, hi = ord_to_f32(ord_u32(mx) + 1u);
      int clo = nv, chi = 0;
      const bool finite = mx < INFINITY && mn > -INFINITY;
      if (finite) {
        for (int it = 0; it < 24 && clo != k_eff; ++it) {
          float f = it < 2 ? 0.5f : ((float)(clo - k_eff) + 0.5f) * __builtin_amdgcn_rcpf((float)(clo - chi));
          f = __builtin_amdgcn_fmed3f(f, 0.125f, 0.875f);
          const float t = uniform(fmaf(hi - lo, f, lo));
          if (!(t > lo && t < hi)) break;  // nothing between the bounds, or their distance overflows
          // the comparisons first, each into scalar registers of its own, then the counts:
          // one after the other they would wait on each other through one register
          uint64_t ge[E];
          int c = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) ge[e] = __builtin_amdgcn_ballot_w64(s[e] >= t);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < E; ++e) c += (int)__popcll(ge[e]);
          if (c >= k_eff) {
            lo = t;
            clo = c;
          } else {
            hi = t;
            chi = c;
          }
        }
      }
      uint64_t take[E];  // lanes whose element e is selected
      float m = mx, low = lo;  // the row's largest score, a lower bound of the selected ones
      if (finite && clo == k_eff) {
#pragma unroll
        for (int e = 0; e < E; ++e) take[e] = __builtin_amdgcn_ballot_w64(s[e] >= lo);
      } else {
        // ties at the k-th score, or scores that are not finite: the same search on the
        // order-preserving keys (0: no valid key), which ends at two neighbouring keys
        uint32_t u[E], top = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          u[e] = key_of(e) < nv ? max(ord_u32(s[e]), 1u) : 0u;
          top = max(top, u[e]);
        }
        m = ord_to_f32(wave_extreme_u32_full<true>(top));
        uint32_t ulo = finite ? ord_u32(lo) : 1u, uhi = finite ? ord_u32(hi) : 0u;  // 0 stands for 2^32
        while (clo != k_eff && uhi - ulo > 1) {
          const uint32_t t = ulo + (uhi - ulo) / 2;
          int c = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) c += (int)__popcll(__builtin_amdgcn_ballot_w64(u[e] >= t));
          if (c >= k_eff) {
            ulo = t;
            clo = c;
          } else {
            uhi = t;
            chi = c;
          }
        }
        low = ord_to_f32(ulo);
        // every key above ulo, and of those equal to it the first by index (all of them
        // where exactly k are left)
        int ties = clo == k_eff ? nv : k_eff - chi;
#pragma unroll
        for (int c = 0; c < E / 4; ++c) {
          uint64_t eq[4];
          int pos = 0, all = 0;  // ties of this chunk in lower lanes, in the whole chunk
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            eq[q] = __builtin_amdgcn_ballot_w64(u[4 * c + q] == ulo);
            pos += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(eq[q] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq[q], 0u));
            all += (int)__popcll(eq[q]);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bool e = u[4 * c + q] == ulo;
            take[4 * c + q] = __builtin_amdgcn_ballot_w64(u[4 * c + q] > ulo || (e && pos < ties));
            pos += e ? 1 : 0;
          }
          ties -= all;
        }
      }
      if (a.scratch && mode == 0) {
        uint64_t* sc = scratch + wave * a.scratch;
        int base = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const uint64_t bal = take[e];
          const int pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
          if (__builtin_amdgcn_inverse_ballot_w64(bal)) sc[pos] = make_key(s[e], (uint32_t)key_of(e));
          base += (int)__popcll(bal);
        }
        wave_sync_lds();
        const int64_t o = (bh * a.Lq + i) * a.k;
        int32_t* ip = a.idx_out ? a.idx_out + o : nullptr;
        float* sp = a.score_out ? a.score_out + o : nullptr;
        // (6, 15 or 21 steps of the network: 48 causal heads of 1024, d = 64, k 8 162 -> 148 us)
        if (a.k <= 8) rows_sorted_out<1, 8>(sc, k_eff, a.k, ip, sp);
        else if (a.k <= 32) rows_sorted_out<1, 32>(sc, k_eff, a.k, ip, sp);
        else if (a.k <= 64) rows_sorted_out<1>(sc, k_eff, a.k, ip, sp);
        else if (a.k <= 128) rows_sorted_out<2>(sc, k_eff, a.k, ip, sp);
        else rows_sorted_out<4>(sc, k_eff, a.k, ip, sp);
        wave_sync_lds();
      }
      // the weights, 0 where not selected; mode 1 tells unselected keys (-1) from weights of 0
      const float none = mode ? -1.f : 0.f;
      // bf16 values: weights 2^16 times as large (exactly; undone by inv_lds), so that the last
      // bit of any float, 2^-149, is one that the last of its three bf16 numbers can hold
      const float up = F32 || mode ? 1.f : 65536.f;
      float sum = 0.f;
      if (a.act == ACT_SOFTMAX) {
        if ((low - m) * a.c > -126.f) {
#pragma unroll
          for (int e = 0; e < E; ++e) s[e] = __builtin_amdgcn_exp2f((s[e] - m) * a.c);
        } else {  // weights below the smallest normal number, which the instruction alone makes 0
#pragma unroll
          for (int e = 0; e < E; ++e) s[e] = exp2f((s[e] - m) * a.c);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
          s[e] = __builtin_amdgcn_inverse_ballot_w64(take[e]) ? s[e] * up : none;
          sum += fmaxf(s[e], 0.f);
        }
        sum = rows_wave_sum(sum);
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) s[e] = __builtin_amdgcn_inverse_ballot_w64(take[e]) ? fmaxf(s[e], 0.f) * up : none;
        sum = up;
      }
      if (lane == 0) {
        inv_lds[r] = 1.f / sum;
        if (mode == 0) bad_lds[r] = 0;
      }
#pragma unroll
      for (int c = 0; c < E / 4; ++c)
        *(f32x4*)&row[256 * c + 4 * lane] = (f32x4){s[4 * c], s[4 * c + 1], s[4 * c + 2], s[4 * c + 3]};
    }
    __syncthreads();

    if (mode) {  // the rows whose dense sum was not finite: selected keys only
      for (int r = wave; r < TR; r += E) {
        if (i0 + r > last || !bad_lds[r]) continue;
        for (int c0 = lane; c0 < D; c0 += 64) {
          float s = 0.f;
          for (int j = 0; j < nkeys; ++j) {
            const float wt = S[r * LDS_ROW + j];
            if (wt != -1.f) s = fmaf(wt, load_elem<T>(Vh, (int64_t)j * D + c0), s);
          }
          store_elem<T>(a.out, (bh * a.Lq + i0 + r) * D + c0, s * inv_lds[r]);
        }
      }
      return;
    }

    // ---- P V over this wave's 64 keys
    f32x4 o[RT][CPL];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < CPL; ++c) o[r][c] = (f32x4){};
    if (live) {
      if constexpr (F32) {
        // lane group g takes keys 4 g .. 4 g + 3 of each 16, one per instruction
#pragma unroll
        for (int kb = 0; kb < 64; kb += 16) {
          f32x4 p[RT];
#pragma unroll
          for (int r = 0; r < RT; ++r) p[r] = *(const f32x4*)&S[(16 * r + n) * LDS_ROW + key0 + kb + 4 * g];
#pragma unroll
          for (int cp = 0; cp < CPL; cp += CPP) {
            if (D > 64) __builtin_amdgcn_sched_barrier(0);
            float v[4][CPP];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              int j = key0 + kb + 4 * g + e;
              j = j < a.Lk ? j : a.Lk - 1;
              __builtin_memcpy(v[e], __builtin_assume_aligned(Vh + (uint32_t)(j * D + n * CPL + cp), 8), CPP * 4);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int c = 0; c < CPP; ++c)
                  o[r][cp + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[r][e], v[e][c], o[r][cp + c], 0, 0, 0);
          }
        }
      } else {
        // lane group g takes keys 8 g .. 8 g + 7 of each 32; their columns are paired up
        // by byte permutes into the operand's order
#pragma unroll
        for (int kb = 0; kb < 64; kb += 32) {
          bf16x8 p[RT][3];
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const float* pr = &S[(16 * r + n) * LDS_ROW + key0 + kb + 8 * g];
            split3_bf16(*(const f32x4*)pr, *(const f32x4*)(pr + 4), p[r]);
          }
#pragma unroll
          for (int cp = 0; cp < CPL; cp += CPP) {
            if (D > 64) __builtin_amdgcn_sched_barrier(0);  // one part's loads at a time: more would spill more
            uint32_t v[8][CPP / 2];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              int j = key0 + kb + 8 * g + e;
              j = j < a.Lk ? j : a.Lk - 1;
              __builtin_memcpy(v[e], __builtin_assume_aligned(Vh + (uint32_t)(j * D + n * CPL + cp), 4), CPP * 2);
            }
#pragma unroll
            for (int c = 0; c < CPP; ++c) {
              const uint32_t sel = c & 1 ? 0x07060302u : 0x05040100u;
              const int w = c / 2;
              const uint4 vf = make_uint4(__builtin_amdgcn_perm(v[1][w], v[0][w], sel), __builtin_amdgcn_perm(v[3][w], v[2][w], sel),
                                          __builtin_amdgcn_perm(v[5][w], v[4][w], sel), __builtin_amdgcn_perm(v[7][w], v[6][w], sel));
#pragma unroll
              for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int t = 0; t < 3; ++t)
                  o[r][cp + c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p[r][t], __builtin_bit_cast(bf16x8, vf), o[r][cp + c], 0, 0, 0);
            }
          }
        }
      }
    }
    __syncthreads();  // every wave has read its weights: the partial sums take their place
    // lane: rows 16 r + 4 g + v, column n * CPL + c; [wave][r][c][lane] as four floats
    f32x4* red = (f32x4*)sm;
    constexpr int HALF = E / 2, PART = RT * CPL * 64;
    static_assert(HALF * PART * 16 <= TR * LDS_ROW * 4, "half the waves' partial sums fit the score tile");
    if (wave >= HALF) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CPL; ++c) red[(wave - HALF) * PART + (r * CPL + c) * 64 + lane] = o[r][c];
    }
    __syncthreads();
    if (wave < HALF) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          f32x4* p = &red[wave * PART + (r * CPL + c) * 64 + lane];
          *p = o[r][c] + *p;
        }
    }
    __syncthreads();
    bool bad = false;
    for (int t = tid; t < RT * 256; t += 64 * E) {
      const int r = t >> 8, l = (t & 255) >> 2, v = t & 3;  // row tile, lane, row of the lane's four
      const int lr = 16 * r + 4 * (l >> 4) + v;
      if (i0 + lr > last) continue;
      float x[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < HALF; ++q) s += ((const float*)&red[q * PART + (r * CPL + c) * 64 + l])[v];
        x[c] = s * inv_lds[lr];
      }
      bool fin = true;
#pragma unroll
      for (int c = 0; c < CPL; ++c) fin = fin && fabsf(x[c]) < INFINITY;
      if (!fin) {
        bad_lds[lr] = 1;
        bad = true;
      }
      T* dst = (T*)a.out + (bh * a.Lq + i0 + lr) * D + (l & 15) * CPL;
      if constexpr (F32) {
        __builtin_memcpy(__builtin_assume_aligned(dst, 8), x, CPL * 4);
      } else {
        uint32_t y[CPL / 2];
#pragma unroll
        for (int c = 0; c < CPL / 2; ++c) y[c] = pack_bf16(x[2 * c], x[2 * c + 1]);
        __builtin_memcpy(__builtin_assume_aligned(dst, 4), y, CPL * 2);
      }
    }
    if (!__syncthreads_or(bad)) return;
  }
}

template <typename T, int D, int E, int TR>
hipError_t launch_rows_inst(RowsArgs a, int64_t BH, hipStream_t st) {
  const size_t sh = (size_t)TR * (64 * E + 4) * 4 + (size_t)E * a.scratch * 8;
  const int64_t grid = BH * a.tiles_per_head;
  constexpr int64_t most = (int64_t(1) << 32) / (64 * E) - 8;  // a launch has fewer than 2^32 threads
  hipError_t e = hipSuccess;
  for (a.first = 0; a.first < grid && e == hipSuccess; a.first += most) {
    const int64_t left = grid - a.first;
    k_rows<T, D, E, TR><<<(unsigned)(left < most ? left : most), 64 * E, sh, st>>>(a);
    e = hipGetLastError();
  }
  return e;
}

template <typename T, int D>
hipError_t launch_rows_d(RowsArgs a, int64_t BH, hipStream_t st) {
  // 32 rows per workgroup halve the reads of keys and values (also where their 128
  // registers spill: bf16 d = 96 6 to 20 of them, d = 128 36 to 39, fp32 d = 128 11 to 29, beside
  // 66 to 94 scalar registers kept in vector lanes everywhere. 96 heads of 512, d = 128, 104 us
  // against 117 with 16 rows and no spill; of 1024, d = 96, 279 against 348); 16 give twice the
  // workgroups where 32 would leave CUs idle (fewer than two workgroups for each of the
  // 256), and where 32 rows and the sort scratch would not fit the 160 KB of LDS, or would leave
  // one workgroup of eight waves a CU (96 heads of 512, k = 200, with the cache outputs, d = 64 241
  // us, where k = 128 takes 115)
  bool tr16 = BH * ((a.Lq + 31) / 32) < 512;
  if (a.Lk > 256 && a.scratch > 128) tr16 = true;
  a.tiles_per_head = tr16 ? (a.Lq + 15) / 16 : (a.Lq + 31) / 32;
  if (a.Lk <= 256) return tr16 ? launch_rows_inst<T, D, 4, 16>(a, BH, st) : launch_rows_inst<T, D, 4, 32>(a, BH, st);
  if (a.Lk <= 512) return tr16 ? launch_rows_inst<T, D, 8, 16>(a, BH, st) : launch_rows_inst<T, D, 8, 32>(a, BH, st);
  return tr16 ? launch_rows_inst<T, D, 16, 16>(a, BH, st) : launch_rows_inst<T, D, 16, 32>(a, BH, st);
}

hipError_t launch_rows(const Problem& pb, hipStream_t st) {
  RowsArgs a;
  a.Q = pb.Q;
  a.K = pb.K;
  a.V = pb.V;
  a.out = pb.out;
  a.Lq = pb.Lq;
  a.tiles_per_head = a.first = 0;
  a.kv_head_stride = pb.kv_head_stride;
  a.Lk = (int)pb.Lk;
  a.k = (int)pb.k;
  a.causal = pb.causal;
  a.act = pb.act;
  a.c = pb.scale * 1.4426950408889634f;
  a.idx_out = pb.idx_out;
  a.score_out = pb.score_out;
  a.scratch = 0;
  if (pb.idx_out || pb.score_out)
    for (a.scratch = 1; a.scratch < pb.k;) a.scratch <<= 1;
#define TOPK_ROWS(T_)                                        \
  switch (pb.d) {                                            \
    case 32: return launch_rows_d<T_, 32>(a, pb.BH, st);     \
    case 64: return launch_rows_d<T_, 64>(a, pb.BH, st);     \
    case 96: return launch_rows_d<T_, 96>(a, pb.BH, st);     \
    case 128: return launch_rows_d<T_, 128>(a, pb.BH, st);   \
    default: return hipErrorInvalidValue;                    \
  }
  if (pb.dtype == T_BF16) TOPK_ROWS(uint16_t)
  TOPK_ROWS(float)
#undef TOPK_ROWS
}

}  // namespace topk
