// Few queries per head against many keys (bf16): their scores and their select.
//
// Heads of at most FEW_ROWS queries (bf16): the scan and the filtered GEMM walk all of a
// head's keys in workgroups made for 128 to 256 queries, a handful of workgroups that use a
// few of their lanes. Here the keys are spread instead: one wave scores 64 keys against up
// to 64 queries (16 x 16 blocks, operands straight from global memory), writes the scores
// and the maximum of every 16 keys (as an order-preserving key). The k-th largest of a
// row's maxima is a bound below which no top-k score lies, since k blocks hold one at or
// above it; the select reads the maxima, then only the blocks that reach the bound (a little
// over k of them).
// Scores: bound by reading the keys once (64 heads of 20001 keys, d = 128, 5 queries: 328 MB
// and 25 MB of scores in 78 us, 4.5 TB/s; the scan took 408), with more queries by writing
// the scores. Select: latency, 20 us a row whatever the number of rows up to a few thousand.
#include "topk_select.h"

#include <math.h>

#include <type_traits>

namespace topk {

template <int RT, int KT>
__global__ __launch_bounds__(256, RT <= 2 ? 4 : 2) void k_few_scores(Problem pb, Pass ps, PassBufs bufs) {
  constexpr int NS = 16 / KT;  // 32-feature steps whose keys are in flight together
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 15, g = lane >> 4;
  if (blockIdx.x == 0 && threadIdx.x == 0) *bufs.redo_count = 0;  // for the select
  // key ranges fastest (consecutive ones on one XCD), then groups of 16 RT queries, then chunks
  const int64_t NG = gridDim.x, bid = blockIdx.x;
  int64_t wg = (NG % 8 == 0) ? (bid % 8) * (NG / 8) + bid / 8 : bid;
  const int64_t nk = (pb.Lk + 64 * KT - 1) / (64 * KT), nq = (pb.C + 16 * RT - 1) / (16 * RT);
  const int64_t key0 = (wg % nk) * (64 * KT) + wave * (16 * KT);
  wg /= nk;
  const int r0 = (int)(wg % nq) * 16 * RT;
  const int64_t cl = wg / nq, id = ps.c0 + cl, bh = id / ps.nchunk, i0 = (id - bh * ps.nchunk) * pb.C;
  const int rows = (int)(pb.Lq - i0 < pb.C ? pb.Lq - i0 : pb.C);  // the chunk's
  if (key0 >= pb.Lk || r0 >= rows) return;
  const uint16_t* Kh = (const uint16_t*)pb.K + bh * pb.kv_head_stride + key0 * pb.d;
  const uint16_t* Qh = (const uint16_t*)pb.Q + (bh * pb.Lq + i0) * pb.d;
  const int d = (int)pb.d, left = (int)(pb.Lk - key0 < 16 * KT ? pb.Lk - key0 : 16 * KT);
  uint32_t ko[KT], qo[RT];
#pragma unroll
  for (int t = 0; t < KT; ++t) ko[t] = (uint32_t)(min(16 * t + n, left - 1) * d + 8 * g);  // past the end: the last key
#pragma unroll
  for (int r = 0; r < RT; ++r) qo[r] = (uint32_t)(min(r0 + 16 * r + n, rows - 1) * d + 8 * g);
  f32x4 acc[KT][RT];
#pragma unroll
  for (int t = 0; t < KT; ++t)
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[t][r] = (f32x4){};
  // 32 features a step, lane group g taking 8 g .. 8 g + 7
  for (int f0 = 0; f0 < d; f0 += 32 * NS) {
    bf16x8 kf[NS][KT];
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (f0 + 32 * s < d)
#pragma unroll
        for (int t = 0; t < KT; ++t) kf[s][t] = *(const bf16x8*)(Kh + ko[t] + f0 + 32 * s);
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (f0 + 32 * s < d) {
        bf16x8 qf[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) qf[r] = *(const bf16x8*)(Qh + qo[r] + f0 + 32 * s);
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
          for (int r = 0; r < RT; ++r) acc[t][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][t], qf[r], acc[t][r], 0, 0, 0);
      }
  }
  // lane: query n of row block r, keys 4 g .. 4 g + 3 of key block t
  const int64_t ld = few_row_len(pb.Lk), nb = ld / 16;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int row = r0 + 16 * r + n;
    const int64_t p = cl * pb.C + row;
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      uint32_t m = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (16 * t + 4 * g + u < left) m = max(m, ord_u32(acc[t][r][u]));
      m = max(m, (uint32_t)__shfl_xor((int)m, 16, 64));
      m = max(m, (uint32_t)__shfl_xor((int)m, 32, 64));
      if (row < rows && 16 * t < left) {  // the row's last block is padded: its extra scores are never read as keys
        *(f32x4*)(bufs.scores + p * ld + key0 + 16 * t + 4 * g) = acc[t][r];
        if (g == 0) bufs.blk[p * nb + key0 / 16 + t] = m;
      }
    }
  }
}

// One wave per row, 64 E >= blocks; rows whose bound lets too many blocks or scores
// through (many equal scores) go to the redo list. CAP: candidates held, KCAP >= k.
template <int E, int KCAP>
__global__ __launch_bounds__(64) void k_few_select(Problem pb, Pass ps, PassBufs bufs) {
  constexpr int CAP = 4 * KCAP;
  __shared__ uint64_t cbuf[CAP];  // candidates; the final sort reuses its start
  __shared__ uint32_t hist[256];
  __shared__ uint16_t blist[CAP];
  const int64_t p = blockIdx.x;
  const RowRef rr = row_of(pb, ps, p);
  if (!rr.ok) return;
  const int lane = threadIdx.x & 63;
  const int k = (int)pb.k, nb = (int)(few_row_len(pb.Lk) / 16);
  const uint32_t* bm = bufs.blk + p * nb;
  uint32_t u[E], mx = 0, mn = 0xFFFFFFFFu;
#pragma unroll
  for (int e = 0; e < E; ++e) u[e] = lane + 64 * e < nb ? bm[lane + 64 * e] : 0u;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    mx = max(mx, u[e]);
    if (lane + 64 * e < nb) mn = min(mn, u[e]);
  }
  // a bound that k to k + k / 8 + 4 blocks reach (or, among equal maxima, more): halving by
  // value, by key where that ends between two keys or after 24 steps
  const uint32_t top = wave_extreme_u32_full<true>(mx);
  uint32_t lo = wave_extreme_u32_full<false>(mn), hi = top + 1;
  int clo = nb;
  const int enough = k + k / 8 + 4;
  if (nb < k) lo = 0;  // fewer blocks than k (at most 1024 keys, which the candidates hold): every key
  for (int it = 0; clo > enough && hi - lo > 1; ++it) {
    uint32_t t = lo + (hi - lo) / 2;
    if (it < 24) {
      const float fl = ord_to_f32(lo), fh = ord_to_f32(hi - 1);
      const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)ord_u32(fmaf(fh - fl, 0.5f, fl)));
      t = v > lo && v < hi ? v : t;
    }
    uint64_t ge[E];
    int c = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) ge[e] = __builtin_amdgcn_ballot_w64(u[e] >= t);
#pragma unroll
    for (int e = 0; e < E; ++e) c += (int)__popcll(ge[e]);
    if (c >= k) {
      lo = t;
      clo = c;
    } else {
      hi = t;
    }
  }
  bool redo = clo > CAP;
  uint32_t c = 0;
  if (!redo) {
    int base = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint64_t m = __builtin_amdgcn_ballot_w64(u[e] >= lo && lane + 64 * e < nb);
      const int pos = base + (int)lanes_below(m);
      if (u[e] >= lo && lane + 64 * e < nb) blist[pos] = (uint16_t)(lane + 64 * e);
      base += (int)__popcll(m);
    }
    wave_sync_lds();
    // 16 blocks at a time, four lanes a block; four such loads in flight
    const float* row = bufs.scores + p * few_row_len(pb.Lk);
    constexpr int U = 4;
    for (int i0 = 0; i0 < clo; i0 += 16 * U) {
      f32x4 x[U];
      int key[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int i = i0 + 16 * q + (lane >> 2);
        key[q] = 16 * (int)blist[i < clo ? i : 0] + 4 * (lane & 3);
        x[q] = *(const f32x4*)(row + key[q]);
        if (i >= clo) key[q] = 0x7FFFFFF0;
      }
#pragma unroll
      for (int q = 0; q < U; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const bool in = key[q] + v < pb.Lk && ord_u32(x[q][v]) >= lo;
          const uint64_t m = __builtin_amdgcn_ballot_w64(in);
          const uint32_t pos = c + lanes_below(m);
          if (in && pos < (uint32_t)CAP)
            cbuf[pos] = ((uint64_t)__float_as_uint(x[q][v]) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)(key[q] + v));
          c += (uint32_t)__popcll(m);
        }
    }
    redo = c > (uint32_t)CAP;
  }
  if (redo) {
    if (lane == 0) bufs.redo_list[atomicAdd(bufs.redo_count, 1)] = (int32_t)p;
    return;
  }
  uint64_t* out = bufs.sel + p * pb.k;
  auto select = [&](auto tag) {
    constexpr int F = decltype(tag)::value;
    uint64_t key[F];
#pragma unroll
    for (int e = 0; e < F; ++e) key[e] = (uint32_t)(lane + 64 * e) < c ? raw_to_key(cbuf[lane + 64 * e]) : 0ull;
    __syncthreads();  // the sort's buffer is the candidates' own
    wave_select_store<F, KCAP>(key, (int)c, (uint32_t)k, k, cbuf, hist, out);
  };
  wave_sync_lds();
  if (c <= 192) select(std::integral_constant<int, 3>{});
  else if (c <= 384) select(std::integral_constant<int, 6>{});
  else if (KCAP <= 256 || c <= 1024) select(std::integral_constant<int, 16>{});
  else select(std::integral_constant<int, CAP / 64>{});
}

hipError_t launch_few_scores(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st) {
  const int RT = pb.C <= 16 ? 1 : pb.C <= 32 ? 2 : 4;
  const int64_t nq = (pb.C + 16 * RT - 1) / (16 * RT) * ps.nc;
  // 64 keys a wave, or 16 (more of their features in flight) where that would leave fewer
  // than two waves a CU: 24 tokens, d_model 768, d_ff 16384 (256 or 1024 waves) 24 -> 16 us;
  // 8 tokens, 1024, 65536 (1024 or 4096 waves) 30 -> 33 us
  const int KT = (pb.Lk + 63) / 64 * nq < 512 ? 1 : 4;
  const int64_t g = ((pb.Lk + 64 * KT - 1) / (64 * KT)) * nq;
  if (g > 0x7FFFFFFF || pb.dtype != T_BF16 || pb.d % 32 != 0 || !b.blk) return hipErrorInvalidValue;
#define TOPK_FEW(RT_)                                                                 \
  do {                                                                                \
    if (KT == 1) k_few_scores<RT_, 1><<<(unsigned)g, 256, 0, st>>>(pb, ps, b);        \
    else k_few_scores<RT_, 4><<<(unsigned)g, 256, 0, st>>>(pb, ps, b);                \
  } while (0)
  if (RT == 1) TOPK_FEW(1);
  else if (RT == 2) TOPK_FEW(2);
  else TOPK_FEW(4);
#undef TOPK_FEW
  return hipGetLastError();
}

hipError_t launch_few_select(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st) {
  const int64_t nb = few_row_len(pb.Lk) / 16;
  const unsigned g = (unsigned)(ps.nc * pb.C);
  if (nb > 4096 || pb.k > 512) return hipErrorInvalidValue;
#define TOPK_FEW(E_)                                                              \
  do {                                                                            \
    if (pb.k <= 256) k_few_select<E_, 256><<<g, 64, 0, st>>>(pb, ps, b);          \
    else k_few_select<E_, 512><<<g, 64, 0, st>>>(pb, ps, b);                      \
  } while (0)
  if (nb <= 512) TOPK_FEW(8);
  else if (nb <= 1024) TOPK_FEW(16);
  else if (nb <= 2048) TOPK_FEW(32);
  else TOPK_FEW(64);
#undef TOPK_FEW
  return launch_tile_redo(pb, ps, b, few_row_len(pb.Lk), st);
}

}  // namespace topk
