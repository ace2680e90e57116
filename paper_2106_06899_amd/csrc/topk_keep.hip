// The candidate select of the filtered path's scan, whose lists need no sort. (In a source of
// its own: the sorting selects, sharing its helpers, otherwise compile to more registers.)
#include "topk_select.h"

#include <math.h>

#include <type_traits>

namespace topk {

// Lists whose order does not depend on scheduling (the filtered path's scan appends each in
// key order): the selection is stored in the order of the lists, which the finalize then
// sums in, and no sort is needed; the debug outputs, which are sorted, are written here.
// The k-th score is found by counting (ballots) the scores at or above a threshold
// between bounds that hold more and fewer than k: first where an exponential tail from the
// smallest candidate (n) to the largest (1) would hold k, then by interpolation; a threshold
// that leaves exactly k ends it, after about five steps of E comparisons. Ties at the k-th
// score and scores that are not finite take the radix select on the full order.
// 64 causal heads of 8192, d = 128, k = 128 (about 340 candidates): 755 -> 489 us against the
// radix select and the sort. (With the sort, the search is no faster than the radix
// select: its counts wait on each other. 16 heads of 32768, k = 64, 180 candidates: 477
// against 445 us; 16384 tokens, 512 of 700: 172 against 134.)
// FULL: n > 64 (E - 1), so that only the last register is partly filled.
template <int E, int KCAP, bool FULL>
__device__ __forceinline__ void cand_select_keep(const Problem& pb, int64_t grow, const uint64_t* b0, const uint64_t* b1,
                                                 int c0, int n, uint32_t k_eff, uint64_t* sbuf, uint32_t* hist,
                                                 uint64_t* out) {
  const int lane = threadIdx.x & 63;
  const int64_t k = pb.k;
  auto in = [&](int e) { return (FULL && e < E - 1) || lane + 64 * e < n; };
  uint64_t wd[E];
  float s[E], mx = -INFINITY, mn = INFINITY;
  if (c0 >= n) {
#pragma unroll
    for (int e = 0; e < E; ++e) wd[e] = b0[FULL && e < E - 1 ? lane + 64 * e : min(lane + 64 * e, n - 1)];
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = FULL && e < E - 1 ? lane + 64 * e : min(lane + 64 * e, n - 1);
      wd[e] = *(i < c0 ? b0 + i : b1 + (i - c0));
    }
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const float x = __uint_as_float((uint32_t)(wd[e] >> 32));
    s[e] = in(e) ? x : -INFINITY;
    mx = __builtin_elementwise_maximum(mx, s[e]);
    mn = __builtin_elementwise_minimum(mn, in(e) ? x : INFINITY);
  }
  mx = wave_extreme_f32_full<true>(mx);
  mn = wave_extreme_f32_full<false>(mn);
  float lo = mn, hi = mx;
  int clo = n, chi = 0;
  const int kk = (int)k_eff;
  const bool finite = mx < INFINITY && mn > -INFINITY;
  if (finite && clo != kk) {
    // log2(n / k) / log2(n) of the way up
    float f = 1.f - __builtin_amdgcn_logf((float)kk) * __builtin_amdgcn_rcpf(__builtin_amdgcn_logf((float)n));
    for (int it = 0; it < 20; ++it) {
      const float t = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(fmaf(hi - lo, __builtin_amdgcn_fmed3f(f, 0.0625f, 0.9375f), lo))));
      if (!(t > lo && t < hi)) break;
      uint64_t ge[E];
      int c = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) ge[e] = __builtin_amdgcn_ballot_w64(s[e] >= t);
#pragma unroll
      for (int e = 0; e < E; ++e) c += (int)__popcll(ge[e]);
      if (c >= kk) {
        lo = t;
        clo = c;
      } else {
        hi = t;
        chi = c;
      }
      if (clo == kk) break;
      f = ((float)(clo - kk) + 0.5f) * __builtin_amdgcn_rcpf((float)(clo - chi));
    }
  }
  uint64_t take[E];
  if (finite && clo == kk) {
#pragma unroll
    for (int e = 0; e < E; ++e) take[e] = __builtin_amdgcn_ballot_w64(s[e] >= lo);
  } else {
    uint64_t key[E];
#pragma unroll
    for (int e = 0; e < E; ++e) key[e] = raw_to_key(wd[e]);
    int shift;
    uint64_t prefix;
    wave_radix_select<E>(key, n, k_eff, hist, &shift, &prefix);
#pragma unroll
    for (int e = 0; e < E; ++e) take[e] = __builtin_amdgcn_ballot_w64(in(e) && (key[e] >> shift) >= (prefix >> shift));
  }
  int base = 0;
  const bool outputs = pb.idx_out || pb.score_out;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int pos = base + (int)lanes_below(take[e]);
    if (__builtin_amdgcn_inverse_ballot_w64(take[e]) && pos < KCAP) {
      const uint64_t w = raw_to_key(wd[e]);
      out[pos] = w;
      if (outputs) sbuf[pos] = w;
    }
    base += (int)__popcll(take[e]);
  }
  for (int64_t t = kk + lane; t < k; t += 64) out[t] = 0ull;
  if (!outputs) return;
  wave_sync_lds();
  auto sort = [&](auto tag) {
    constexpr int P = decltype(tag)::value;
    uint64_t r[P];
#pragma unroll
    for (int e = 0; e < P; ++e) r[e] = e * 64 + lane < kk ? sbuf[e * 64 + lane] : 0ull;
    wave_sort_desc<P>(r);
#pragma unroll
    for (int e = 0; e < P; ++e) sbuf[e * 64 + lane] = r[e];
  };
  if (kk <= 128) sort(std::integral_constant<int, 2>{});
  else if (KCAP <= 256 || kk <= 256) sort(std::integral_constant<int, 4>{});
  else sort(std::integral_constant<int, (KCAP > 256 ? 8 : 4)>{});
  wave_sync_lds();
  write_selection(pb, grow, k_eff, lane, 64, [&](int64_t t) { return sbuf[t]; });
}

// BIG: rows of up to 2048 candidates and k <= 512. A row whose lists overflowed or hold fewer
// than k_eff keys goes to the redo list.
template <bool BIG>
__global__ __launch_bounds__(64) void k_keep_select(Problem pb, Pass ps, PassBufs bufs) {
  __shared__ uint64_t sbuf[BIG ? 512 : 256];
  __shared__ uint32_t hist[256];
  __shared__ uint32_t misc[8];
  const int64_t p = blockIdx.x;
  constexpr int KCAP = BIG ? 512 : 256, NMAX = BIG ? 128 * CAND_REGS : 64 * CAND_REGS;
  const RowRef rr = row_of(pb, ps, p);
  if (!rr.ok) return;
  const int64_t nv = valid_keys(pb, rr.i);
  const uint32_t k_eff = (uint32_t)(pb.k < nv ? pb.k : nv);
  const int64_t c0 = bufs.cnt[2 * p], c1 = bufs.cnt[2 * p + 1];
  if (c0 > bufs.caph || c1 > bufs.caph || c0 + c1 < (int64_t)k_eff || k_eff > KCAP || c0 + c1 > NMAX) {
    if ((threadIdx.x & 63) == 0) bufs.redo_list[atomicAdd(bufs.redo_count, 1)] = (int32_t)p;
    return;
  }
  const int n = (int)(c0 + c1);
  const uint64_t* b0 = bufs.cand + (2 * p) * bufs.caph;
  uint64_t* out = bufs.sel + p * pb.k;
  const int64_t grow = rr.bh * pb.Lq + rr.i;
  auto keep = [&](auto regs, auto full) {
    cand_select_keep<decltype(regs)::value, KCAP, decltype(full)::value>(pb, grow, b0, b0 + bufs.caph, (int)c0, n, k_eff, sbuf, hist, out);
  };
  using std::integral_constant;
  if (BIG) {
    if (n <= 512) keep(integral_constant<int, 8>{}, std::false_type{});
    else if (n <= 1024) keep(integral_constant<int, CAND_REGS>{}, std::false_type{});
    else keep(integral_constant<int, 2 * CAND_REGS>{}, std::false_type{});
  } else if (n <= 128) keep(integral_constant<int, 2>{}, std::false_type{});
  else if (n <= 192) keep(integral_constant<int, 3>{}, std::true_type{});
  else if (n <= 256) keep(integral_constant<int, 4>{}, std::true_type{});
  else if (n <= 320) keep(integral_constant<int, 5>{}, std::true_type{});
  else if (n <= 384) keep(integral_constant<int, 6>{}, std::true_type{});
  else if (n <= 448) keep(integral_constant<int, 7>{}, std::true_type{});
  else if (n <= 512) keep(integral_constant<int, 8>{}, std::true_type{});
  else {
    auto getkey = [&](int64_t e) { return raw_to_key(e < c0 ? b0[e] : b0[bufs.caph + (e - c0)]); };
    team_topk<64>(getkey, n, k_eff, (uint32_t)pb.k, sbuf, pow2_at_least(k_eff), hist, misc, out);
    write_selection(pb, grow, k_eff, threadIdx.x, 64, [&](int64_t t) { return sbuf[t]; });
  }
}

hipError_t launch_keep_select(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st) {
  const unsigned g = (unsigned)(ps.nc * pb.C);
  if (b.cand_single) return hipErrorInvalidValue;
  if (b.caph > 512) k_keep_select<true><<<g, 64, 0, st>>>(pb, ps, b);
  else k_keep_select<false><<<g, 64, 0, st>>>(pb, ps, b);
  return hipGetLastError();
}

}  // namespace topk
