// Backward pass by cells (Section 2.2's backward pseudo-code, where the rows keep a large
// enough share of the keys): the selected (row, key) pairs of every 64-row strip are
// grouped by 64-key cell, and the gradients are matrix products whose sparse operand is
// expanded in LDS, cell by cell:
//  1. k_cells_build: the strip's pairs in cell order (entry = local row, local key) with
//     their weights, recomputed from the cached scores, and each cell's range;
//  2. d_top_actv = d_out . V[j]: the score GEMM on d_out and V, whose tiles stay on chip
//     and give each pair its entry (k_tile_scores_mfma<3>); a ReLU's gate is applied there;
//  3. k_cells_vjp: the softmax backpropagated to the score gradients;
//  4. k_cells_mm: d_Q = D K, d_K = D^T Q, d_V = P^T d_out, with D and P the sparse
//     matrices of score gradients and weights.
// The products read a value, key or query row once per 128 rows or keys of the other
// side, where the gathers of the list kernels read four rows per pair: at 16384 tokens,
// d_model 768, 512 of 4096 units kept, 51 GB. No matrix of the size of the scores is
// stored, and every sum runs in a fixed order (the order of a cell's list, which is not
// fixed, only says where its values go).
//
// The sparse operand keeps its 32 bits: it lies in LDS as floats, and each wave takes the
// values apart into three bf16 numbers that add up to them exactly, so that a product differs
// from a gather's only by the order of its 32-bit sums: 48 heads of 1024, d = 64, 2.0e-4 of
// d_K's stored values are not the 64-bit result rounded, by the gathers 1.7e-4 (by two bf16
// numbers, 16 or 17 bits: 2.4e-3, and the step of 16384 tokens below takes 2040 us for 2425).
// A result that is not finite (an infinite or NaN row that a zero met) is computed again for
// its row alone, from its own pairs.
//
// Bound by latency (two waves a SIMD: 70 KB of LDS a workgroup) and, for wide rows, by the
// matrix instructions and the taking apart, about 45 vector instructions per 12 of them. Whole
// backward pass, lists -> cells: 16384 tokens, d_model 768, 512 of 4096 units: 5260 -> 1445 us;
// of 16384: 6220 -> 4120; 48 heads of 1024 tokens, d = 64, k = 64: 247 -> 215; 32 heads of 2048,
// d = 128, k = 128: 717 -> 556 (causal 719 -> 582).
#include "topk_device.h"
#include "topk_internal.h"

#include <math.h>

namespace topk {

// A workgroup barrier for LDS alone: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One workgroup per strip; cells <= CELL_MAX (one thread each in the scan). A strip in which
// a row lists a key twice is marked (after its ranges), and its lists are in pair order: the
// products then add its entries one by one instead of storing them side by side.
__global__ __launch_bounds__(1024) void k_cells_build(BwdProblem bp, CellBufs cb) {
  extern __shared__ uint32_t seen[];  // cb.seen words: a bit per (row, key) of the strip
  __shared__ uint32_t cnt[CELL_MAX];
  __shared__ uint32_t wsum[16], repeated;
  __shared__ float mx_lds[64], inv_lds[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t strip = blockIdx.x, bh = strip / cb.nstrip, r0 = (strip - bh * cb.nstrip) * 64;
  const int nrows = (int)(bp.Lq - r0 < 64 ? bp.Lq - r0 : 64);
  const int64_t base = (bh * bp.Lq + r0) * bp.k;
  const uint32_t k = (uint32_t)bp.k, n = (uint32_t)nrows * k;
  const int32_t* idx = bp.idx + base;
  const float* dots = bp.dots + base;
  auto valid = [&](int32_t j) { return j >= 0 && (int64_t)j < bp.Lk; };
  if (tid < cb.ncell) cnt[tid] = 0;
  if (tid == 0) repeated = 0;
  for (int i = tid; i < cb.seen; i += 1024) seen[i] = 0;
  __syncthreads();
#pragma unroll 4
  for (uint32_t e = tid; e < n; e += 1024) {
    const int32_t j = idx[e];
    if (!valid(j)) continue;
    atomicAdd(&cnt[j >> 6], 1u);
    const uint32_t bit = e / k * (uint32_t)cb.ncell * 64u + (uint32_t)j;
    if (atomicOr(&seen[bit >> 5], 1u << (bit & 31u)) >> (bit & 31u) & 1u) repeated = 1;
  }
  // the softmax's maximum and normaliser of each row, over its cached scores, 16 lanes a row
  const int sr = tid >> 4, sl = tid & 15;
  if (bp.act == ACT_SOFTMAX && sr < nrows) {
    const uint32_t o = (uint32_t)sr * k;
    float mx = -INFINITY, z = 0.f;
#pragma unroll 8
    for (uint32_t m = sl; m < k; m += 16) mx = fmaxf(mx, valid(idx[o + m]) ? dots[o + m] : -INFINITY);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
#pragma unroll 8
    for (uint32_t m = sl; m < k; m += 16) z += valid(idx[o + m]) ? __expf(bp.scale * (dots[o + m] - mx)) : 0.f;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) z += __shfl_xor(z, off, 64);
    if (sl == 0) {
      mx_lds[sr] = mx;
      inv_lds[sr] = 1.f / z;
    }
  }
  __syncthreads();
  const uint32_t c = tid < cb.ncell ? cnt[tid] : 0u;
  const uint32_t incl = wave_incl_scan_full(c);
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  const uint32_t beg = (uint32_t)base + before + incl - c;
  int32_t* off = cb.off + strip * cb.off_row;
  if (tid < cb.ncell) {
    cnt[tid] = beg;
    off[tid] = (int32_t)beg;
    if (tid == cb.ncell - 1) off[cb.ncell] = (int32_t)(beg + c);
  }
  __syncthreads();
  auto store = [&](uint32_t pos, uint32_t e, int32_t j) {
    const uint32_t r = e / k;
    const float s = dots[e];
    cb.ent[pos] = r << 6 | ((uint32_t)j & 63u);
    cb.w[pos] = bp.act == ACT_SOFTMAX ? __expf(bp.scale * (s - mx_lds[r])) * inv_lds[r] : fmaxf(s, 0.f);
  };
  if (!repeated) {
#pragma unroll 4
    for (uint32_t e = tid; e < n; e += 1024) {
      const int32_t j = idx[e];
      if (valid(j)) store(atomicAdd(&cnt[j >> 6], 1u), e, j);
    }
  } else if (wave == 0) {  // in pair order: 64 pairs at a time, lanes of one cell by rank
    for (uint32_t e0 = 0; e0 < n; e0 += 64) {
      const uint32_t e = e0 + lane;
      const int32_t j = e < n ? idx[e] : -1;
      const bool ok = valid(j);
      const uint32_t cell = ok ? (uint32_t)j >> 6 : 0u;
      uint64_t peers = __ballot(ok);
#pragma unroll
      for (int t = 0; t < 8; ++t) {  // (CELL_MAX is 2^8)
        const bool bit = cell >> t & 1u;
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
      }
      const uint32_t rank = lanes_below(peers), first = ok ? cnt[cell] : 0u;
      wave_sync_lds();
      if (ok && rank == 0) cnt[cell] = first + (uint32_t)__popcll(peers);
      wave_sync_lds();
      if (ok) store(first + rank, e, j);
    }
  }
  if (tid == 0) off[cb.ncell + 1] = (int32_t)repeated;
}

// Softmax: the score gradients scale w (a - sum of w a over the row), one workgroup per
// strip; cb.a holds each pair's a = d_out . V[j] and takes its score gradient. The order of
// a cell's pairs is not fixed, so a row's sum is taken in whole numbers: in units of 2^-40
// of the power of two at its largest term (finer than a float sum), which any order adds
// to the same total.
__global__ __launch_bounds__(1024) void k_cells_vjp(BwdProblem bp, CellBufs cb) {
  __shared__ uint32_t top[64];
  __shared__ unsigned long long sum[64];
  __shared__ float gs[64];
  constexpr int U = 8;  // pairs held per thread; longer strips read the rest again each time
  const int tid = threadIdx.x;
  const int32_t* off = cb.off + blockIdx.x * (int64_t)cb.off_row;
  const int32_t beg = off[0], end = off[cb.ncell], more = beg + 1024 * U + tid;
  if (tid < 64) {
    top[tid] = 0;
    sum[tid] = 0;
  }
  uint32_t row[U];
  float w[U], a[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int32_t i = beg + tid + 1024 * u;
    const bool in = i < end;
    row[u] = in ? cb.ent[i] >> 6 : 64u;
    w[u] = in ? cb.w[i] : 0.f;
    a[u] = in ? cb.a[i] : 0.f;
  }
  __syncthreads();
  auto largest = [&](uint32_t r, float wa) { atomicMax(&top[r], __float_as_uint(fabsf(wa))); };
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (row[u] < 64u) largest(row[u], w[u] * a[u]);
  for (int32_t i = more; i < end; i += 1024) largest(cb.ent[i] >> 6, cb.w[i] * cb.a[i]);
  __syncthreads();
  auto unit = [&](uint32_t r) { return 40 - ((int)(top[r] >> 23) - 127); };
  auto term = [&](uint32_t r, float wa) {
    if (top[r] < 0x7F800000u) atomicAdd(&sum[r], (unsigned long long)__double2ll_rn(ldexp((double)wa, unit(r))));
  };
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (row[u] < 64u) term(row[u], w[u] * a[u]);
  for (int32_t i = more; i < end; i += 1024) term(cb.ent[i] >> 6, cb.w[i] * cb.a[i]);
  __syncthreads();
  if (tid < 64) gs[tid] = top[tid] < 0x7F800000u ? (float)ldexp((double)(long long)sum[tid], -unit(tid)) : NAN;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (row[u] < 64u) cb.a[beg + tid + 1024 * u] = bp.scale * w[u] * (a[u] - gs[row[u]]);
  for (int32_t i = more; i < end; i += 1024) cb.a[i] = bp.scale * cb.w[i] * (cb.a[i] - gs[cb.ent[i] >> 6]);
}

// out = X B for every head, X the sparse [M x N] matrix of the cells' values: M = rows and
// N = keys, or (TRANS) M = keys and N = rows. A workgroup owns 128 of M and 64 WC columns
// of B and walks the 64-wide cells of N (a range of them where the products are split).
// Per cell: the listed values are put into a clear tile in LDS (128 x 64), each wave
// multiplies it with its 64 columns of B, and the entries are cleared again while the next
// cell's tile is multiplied. B is read straight from global memory (16 lanes cover a row's 128 contiguous bytes, column
// n * 4 + c is column n of tile c; 16-bit columns are paired up by byte permutes).
struct MmArgs {
  const int32_t* off;
  const uint32_t* ent;
  const float* val[2];
  const void* B[2];
  void* out[2];
  float* part;        // [nsplit][which][BH * M][d] partial sums when nsplit > 1
  int64_t BH, M, N, d, head_m, head_n;  // head strides (elements) of out and B
  int nstrip, ncell, off_row, mtiles, ctiles, nsplit, which;
};

template <bool TRANS>
__device__ void cells_fix_row(const MmArgs& a, int y, int64_t bh, int64_t m) {
  // out row m from its own pairs, by one wave: lanes test 64 entries at a time. A zero score
  // gradient (a closed ReLU gate, say) adds nothing to d_Q, whatever its key holds, as by lists.
  const int lane = threadIdx.x & 63;
  const uint16_t* B = (const uint16_t*)a.B[y] + bh * a.head_n;
  uint16_t* out = (uint16_t*)a.out[y] + bh * a.head_m + m * a.d;
  const int nc = TRANS ? a.nstrip : a.ncell;
  const uint32_t local = (uint32_t)m & 63u;
  for (int64_t c0 = 0; c0 < a.d; c0 += 64) {
    const int64_t col = c0 + lane < a.d ? c0 + lane : 0;
    float s = 0.f;
    for (int c = 0; c < nc; ++c) {
      const int64_t o = TRANS ? (bh * a.nstrip + c) * a.off_row + (m >> 6) : (bh * a.nstrip + (m >> 6)) * a.off_row + c;
      // the cell's values of the row, one column of the cell per lane, then their sum by column
      // (a list's order is not fixed)
      float x = 0.f;
      uint64_t have = 0;
      for (int32_t i0 = a.off[o]; i0 < a.off[o + 1]; i0 += 64) {
        const int32_t i = i0 + lane;
        const bool in = i < a.off[o + 1];
        const uint32_t e = in ? a.ent[i] : 0u;
        const float v = in ? a.val[y][i] : 0.f;
        uint64_t hit = __ballot(in && (TRANS ? (e & 63u) : (e >> 6)) == local && (TRANS || v != 0.f));
        for (; hit; hit &= hit - 1) {
          const int l = __builtin_ctzll(hit);
          const uint32_t el = (uint32_t)__builtin_amdgcn_readlane((int)e, l);
          const float vl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
          const int at = (int)(TRANS ? (el >> 6) : (el & 63u));
          if (lane == at) x += vl;
          have |= uint64_t(1) << at;
        }
      }
      for (; have; have &= have - 1) {
        const int at = __builtin_ctzll(have);
        const float xl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), at));
        s = fmaf(xl, load_elem<uint16_t>(B, ((int64_t)c * 64 + at) * a.d + col), s);
      }
    }
    if (c0 + lane < a.d) store_elem<uint16_t>(out, c0 + lane, s);
  }
}

template <int WC, bool TRANS>
__global__ __launch_bounds__(256, 2) void k_cells_mm(MmArgs a) {
  constexpr int WR = 4 / WC;       // waves along the rows of the tile
  constexpr int RT = 8 / WR;       // 16-row tiles per wave
  // the sparse operand of two cells in turn, in 32 bits
  constexpr int TS = 68, TILE = 128 * TS;  // row stride, elements per tile
  // its values 2^16 times as large (exactly; undone at the end), so that the last bit of any
  // float, 2^-149, is one that the last of its three bf16 numbers can hold
  constexpr float UP = 65536.f;
  __shared__ __attribute__((aligned(16))) float tiles[2][TILE];
  __shared__ int bad_lds[128];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15,
            g = lane >> 4;
  // tiles of M fastest, then heads, then column tiles, then splits, then the two products;
  // contiguous ranges per XCD
  const int64_t NGR = gridDim.x, bid = blockIdx.x;
  int64_t wg = (NGR % 8 == 0) ? (bid % 8) * (NGR / 8) + bid / 8 : bid;
  const int64_t mt = wg % a.mtiles;
  wg /= a.mtiles;
  const int64_t bh = wg % a.BH;
  wg /= a.BH;
  const int ct = (int)(wg % a.ctiles);
  wg /= a.ctiles;
  const int sp = (int)(wg % a.nsplit), y = (int)(wg / a.nsplit);
  const int wc = wave % WC, wr = wave / WC;
  const int ncn = TRANS ? a.nstrip : a.ncell;  // cells along N
  const int c_beg = (int)((int64_t)ncn * sp / a.nsplit), c_end = (int)((int64_t)ncn * (sp + 1) / a.nsplit);
  const float* val = a.val[y];
  const uint16_t* B = (const uint16_t*)a.B[y] + bh * a.head_n;
  const int64_t col0 = (int64_t)(ct * WC + wc) * 64 + n * 4;  // this lane's first column
  const int64_t colr = col0 < a.d ? col0 : 0;                 // columns past d are read as 0 .. 3, not stored
  // a cell's two lists: of both strips of M along N, or (TRANS) of the two neighbouring
  // cells of M in a strip of N
  const int m64 = (int)mt * 2;
  const bool two = m64 + 1 < (TRANS ? a.ncell : a.nstrip);
  f32x4 acc[RT][4];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = (f32x4){};
  for (int i = tid; i < 2 * TILE / 4; i += 256) ((f32x4*)&tiles[0][0])[i] = (f32x4){};
  const uint32_t boff = (uint32_t)(8 * g * a.d + colr);  // this lane's operand rows of a whole cell: 8 g + e of each 32
  // entries of a cell held per thread, read while the cell before is multiplied; the
  // previous cell's, to clear its tile
  constexpr int U = 4;
  uint32_t ee[U], eo[U];
  float vv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) eo[u] = 0xFFFFFFFFu;
  int ob0 = 0, on0 = 0, ob1 = 0, on1 = 0;  // its lists, for the entries not held
  int buf = 0;
  __syncthreads();
  for (int cb0 = c_beg; cb0 < c_end; cb0 += 64) {
    // lane l holds the ranges of cell cb0 + l: n0 entries from b0, then n1 from b1
    int32_t lb0 = 0, ln0 = 0, lb1 = 0, ln1 = 0, lrep = 0;
    if (cb0 + lane < c_end) {
      const int c = cb0 + lane;
      if (TRANS) {
        const int32_t* o = a.off + (bh * a.nstrip + c) * (int64_t)a.off_row + m64;
        lb0 = o[0];
        lb1 = o[1];
        ln0 = lb1 - lb0;
        ln1 = two ? o[2] - lb1 : 0;
        lrep = o[a.ncell + 1 - m64];
      } else {
        const int32_t* o = a.off + (bh * a.nstrip + m64) * (int64_t)a.off_row + c;
        lb0 = o[0];
        ln0 = o[1] - lb0;
        if (two) {
          lb1 = o[a.off_row];
          ln1 = o[a.off_row + 1] - lb1;
        }
        lrep = o[a.ncell + 1 - c] | (two ? o[a.off_row + a.ncell + 1 - c] : 0);
      }
    }
    int32_t b0, n0, b1, n1;
    auto ranges = [&](int l) {
      b0 = __builtin_amdgcn_readlane(lb0, l);
      n0 = __builtin_amdgcn_readlane(ln0, l);
      b1 = __builtin_amdgcn_readlane(lb1, l);
      n1 = __builtin_amdgcn_readlane(ln1, l);
    };
    // entry i of the cell with its list in bit 12
    auto fetch = [&](int i, uint32_t& e, float& v) {
      const int src = i < n0 ? b0 + i : b1 + (i - n0);
      e = a.ent[src] | (i < n0 ? 0u : 4096u);
      v = val[src];
    };
    auto fetch_all = [&](uint32_t (&e)[U], float (&v)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        e[u] = 0xFFFFFFFFu;
        if (tid + 256 * u < n0 + n1) fetch(tid + 256 * u, e[u], v[u]);
      }
    };
    // the entry's place in a tile
    auto place = [&](uint32_t e) {
      const uint32_t r = e >> 6 & 63u, k = e & 63u, h = e >> 12 << 6;
      return TRANS ? (k + h) * TS + r : (r + h) * TS + k;
    };
    auto put = [&](float* t, uint32_t e, float v) { t[place(e)] = v * UP; };
    auto clear = [&](float* t, uint32_t e) { t[place(e)] = 0.f; };
    uint64_t todo = __ballot(ln0 + ln1 > 0);
    const uint64_t rep = __ballot(lrep != 0);  // cells with keys listed twice in a row
    // operand rows of cell c (rows past N repeat the last: their tile columns are 0)
    auto brow = [&](int c, int o, int e) {  // this lane's e-th row from row o on
      const uint16_t* Bc = B + (int64_t)c * 64 * a.d;
      const int jmax = (int)(a.N - 1 - (int64_t)c * 64);
      return jmax >= 63 ? Bc + (o + e) * a.d + boff : Bc + (uint32_t)(min(o + 8 * g + e, jmax) * a.d + colr);
    };
    uint32_t bq[2][8][2];
    auto load_b = [&](int c) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 8; ++e) __builtin_memcpy(bq[kb][e], __builtin_assume_aligned(brow(c, 32 * kb, e), 8), 8);
    };
    if (todo) {
      ranges(__builtin_ctzll(todo));
      fetch_all(ee, vv);
      load_b(cb0 + __builtin_ctzll(todo));
    }
    while (todo) {
      const int c = cb0 + __builtin_ctzll(todo);
      todo &= todo - 1;
      float* cur = tiles[buf];
      buf ^= 1;
      // with registers to spare the next cell's entries are asked for before this cell's
      // are put in place, otherwise after
      const int c0n = n0, c1n = n1, c0b = b0, c1b = b1;
      uint32_t en[U];
      float vn[U];
      if (WC < 4 && todo) {
        ranges(__builtin_ctzll(todo));
        fetch_all(en, vn);
      }
      const int s0n = n0, s1n = n1, s0b = b0, s1b = b1;
      n0 = c0n, n1 = c1n, b0 = c0b, b1 = c1b;
      if (!(rep >> (c - cb0) & 1)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (ee[u] != 0xFFFFFFFFu) put(cur, ee[u], vv[u]);
        for (int i0 = tid + 256 * U; i0 < n0 + n1; i0 += 1024) {  // a cell of more: four loads at a time
          uint32_t e[4];
          float v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int i = i0 + 256 * u;
            fetch(i < n0 + n1 ? i : i0, e[u], v[u]);
            if (i >= n0 + n1) e[u] = 0xFFFFFFFFu;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (e[u] != 0xFFFFFFFFu) put(cur, e[u], v[u]);
        }
      } else if (tid < 128) {  // each thread adds its row's entries, in the lists' order
        for (int i = 0; i < n0 + n1; ++i) {
          uint32_t e;
          float v;
          fetch(i, e, v);
          if ((int)((TRANS ? e & 63u : e >> 6 & 63u) + (e >> 12 << 6)) == tid) cur[place(e)] += v * UP;
        }
      }
      lds_barrier();  // the tile is complete; every wave is done with the other one
      // clear the other tile's entries, then keep this cell's for the next turn
      float* oth = tiles[buf];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (eo[u] != 0xFFFFFFFFu) clear(oth, eo[u]);
        eo[u] = ee[u];
      }
      for (int i0 = tid + 256 * U; i0 < on0 + on1; i0 += 1024) {
        uint32_t e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = i0 + 256 * u < on0 + on1 ? i0 + 256 * u : i0;
          e[u] = a.ent[i < on0 ? ob0 + i : ob1 + (i - on0)] | (i < on0 ? 0u : 4096u);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) clear(oth, e[u]);
      }
      ob0 = b0;
      on0 = n0;
      ob1 = b1;
      on1 = n1;
      if (WC < 4) {
        n0 = s0n, n1 = s1n, b0 = s0b, b1 = s1b;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ee[u] = en[u];
          vv[u] = vn[u];
        }
      } else if (todo) {
        ranges(__builtin_ctzll(todo));
        fetch_all(ee, vv);
      }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          bf16x8 bv[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t sel = q & 1 ? 0x07060302u : 0x05040100u;
            const int w = q / 2;
            bv[q] = __builtin_bit_cast(bf16x8, make_uint4(__builtin_amdgcn_perm(bq[kb][1][w], bq[kb][0][w], sel),
                                                          __builtin_amdgcn_perm(bq[kb][3][w], bq[kb][2][w], sel),
                                                          __builtin_amdgcn_perm(bq[kb][5][w], bq[kb][4][w], sel),
                                                          __builtin_amdgcn_perm(bq[kb][7][w], bq[kb][6][w], sel)));
          }
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const float* o = cur + ((wr * RT + r) * 16 + n) * TS + 32 * kb + 8 * g;
            bf16x8 part[3];
            split3_bf16(*(const f32x4*)o, *(const f32x4*)(o + 4), part);
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
              for (int q = 0; q < 4; ++q) acc[r][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part[p], bv[q], acc[r][q], 0, 0, 0);
          }
        }
      if (todo) load_b(cb0 + __builtin_ctzll(todo));  // the next cell's, while its entries are put in place
      lds_barrier();  // the other tile is clear: the next cell's entries may go there
    }
  }
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] *= 1.f / UP;
  // lane: rows 4 g + v of row tile r, columns col0 .. col0 + 3
  if (a.nsplit > 1) {
    float* part = a.part + ((int64_t)sp * a.which + y) * a.BH * a.M * a.d;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t m = mt * 128 + (wr * RT + r) * 16 + 4 * g + v;
        if (m < a.M && col0 < a.d)
          *(f32x4*)(part + (bh * a.M + m) * a.d + col0) = (f32x4){acc[r][0][v], acc[r][1][v], acc[r][2][v], acc[r][3][v]};
      }
    return;
  }
  for (int i = tid; i < 128; i += 256) bad_lds[i] = 0;
  __syncthreads();
  bool bad = false;
  uint16_t* out = (uint16_t*)a.out[y] + bh * a.head_m;
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int lm = (wr * RT + r) * 16 + 4 * g + v;
      const int64_t m = mt * 128 + lm;
      if (m < a.M && col0 < a.d) {
        const float x0 = acc[r][0][v], x1 = acc[r][1][v], x2 = acc[r][2][v], x3 = acc[r][3][v];
        if (!(fabsf(x0) < INFINITY && fabsf(x1) < INFINITY && fabsf(x2) < INFINITY && fabsf(x3) < INFINITY)) {
          bad_lds[lm] = 1;
          bad = true;
        }
        *(uint2*)(out + m * a.d + col0) = make_uint2(pack_bf16(x0, x1), pack_bf16(x2, x3));
      }
    }
  if (!__syncthreads_or(bad)) return;
  for (int i = wave; i < 128; i += 4)
    if (mt * 128 + i < a.M && bad_lds[i]) cells_fix_row<TRANS>(a, y, bh, mt * 128 + i);
}

// Sums the partial products of split calls in order; one wave per row of M.
template <bool TRANS>
__global__ __launch_bounds__(256) void k_cells_reduce(MmArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t rows = a.BH * a.M, id = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (id >= rows * a.which) return;
  const int y = (int)(id / rows);
  const int64_t row = id - y * rows, bh = row / a.M, m = row - bh * a.M;
  uint16_t* out = (uint16_t*)a.out[y] + bh * a.head_m + m * a.d;
  bool bad = false;
  for (int64_t c = lane * 4; c < a.d; c += 256) {
    f32x4 s = {};
    for (int p = 0; p < a.nsplit; ++p) s += *(const f32x4*)(a.part + (((int64_t)p * a.which + y) * rows + row) * a.d + c);
#pragma unroll
    for (int q = 0; q < 4; ++q) bad = bad || !(fabsf(s[q]) < INFINITY);
    *(uint2*)(out + c) = make_uint2(pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3]));
  }
  if (__ballot(bad)) cells_fix_row<TRANS>(a, y, bh, m);
}

// ------------------------------------------------------------------ launches
static int mm_splits(int64_t wgs, int cells) {
  // enough workgroups for the 256 CUs (two fit each; 700 and 1400 were no faster: the
  // partial sums cost what they save), at least three cells per part
  int s = 1;
  while (s < 8 && wgs * s < 384 && cells / (s + 1) >= 3) ++s;
  return s;
}
static int mm_cols(int64_t d) { return d <= 64 ? 1 : d <= 128 ? 2 : 4; }  // 64-column groups per workgroup

static hipError_t launch_mm(const BwdProblem& bp, const CellBufs& cb, bool trans, hipStream_t st) {
  MmArgs a{};
  a.off = cb.off;
  a.ent = cb.ent;
  a.BH = bp.BH;
  a.d = bp.d;
  a.nstrip = (int)cb.nstrip;
  a.ncell = (int)cb.ncell;
  a.off_row = (int)cb.off_row;
  const int64_t hq = bp.Lq * bp.d, hk = bp.kv_head_stride;
  if (!trans) {  // d_Q = D K
    a.val[0] = cb.a; a.B[0] = bp.K; a.out[0] = bp.dQ;
    a.M = bp.Lq; a.N = bp.Lk; a.head_m = hq; a.head_n = hk; a.which = 1;
  } else {       // d_K = D^T Q, d_V = P^T d_out
    a.val[0] = cb.a; a.B[0] = bp.Q; a.out[0] = bp.dK;
    a.val[1] = cb.w; a.B[1] = bp.dout; a.out[1] = bp.dV;
    a.M = bp.Lk; a.N = bp.Lq; a.head_m = hk; a.head_n = hq; a.which = 2;
  }
  const int WC = mm_cols(bp.d);
  a.mtiles = (int)((a.M + 127) / 128);
  a.ctiles = (int)((bp.d + 64 * WC - 1) / (64 * WC));
  a.nsplit = trans ? cb.split_k : cb.split_q;
  a.part = cb.part;
  const int64_t grid = (int64_t)a.mtiles * a.BH * a.ctiles * a.nsplit * a.which;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
#define TOPK_MM(WC_)                                                                     \
  do {                                                                                   \
    if (trans) k_cells_mm<WC_, true><<<(unsigned)grid, 256, 0, st>>>(a);              \
    else k_cells_mm<WC_, false><<<(unsigned)grid, 256, 0, st>>>(a);                   \
  } while (0)
  if (WC == 1) TOPK_MM(1);
  else if (WC == 2) TOPK_MM(2);
  else TOPK_MM(4);
#undef TOPK_MM
  if (a.nsplit > 1) {
    const unsigned gr = (unsigned)((a.BH * a.M * a.which + 3) / 4);
    if (trans) k_cells_reduce<true><<<gr, 256, 0, st>>>(a);
    else k_cells_reduce<false><<<gr, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

CellLayout cell_layout(const BwdProblem& bp) {
  const int64_t BH = bp.BH, Lq = bp.Lq, Lk = bp.Lk, d = bp.d;
  CellLayout L;
  L.nstrip = (Lq + 63) / 64;
  L.ncell = (Lk + 63) / 64;
  L.off_row = L.ncell + 2;
  const int WC = mm_cols(d);
  const int64_t ct = (d + 64 * WC - 1) / (64 * WC);
  L.split_q = mm_splits((Lq + 127) / 128 * BH * ct, (int)L.ncell);
  L.split_k = mm_splits((Lk + 127) / 128 * BH * ct * 2, (int)L.nstrip);
  const int64_t pq = L.split_q > 1 ? L.split_q * BH * Lq * d : 0, pk = L.split_k > 1 ? 2 * L.split_k * BH * Lk * d : 0;
  L.part_floats = pq > pk ? pq : pk;
  return L;
}

hipError_t launch_backward_cells(const BwdProblem& bp, const CellBufs& cb, hipStream_t st) {
  const int64_t strips = bp.BH * cb.nstrip;
  if (cb.ncell > CELL_MAX || strips > 0x7FFFFFFF) return hipErrorInvalidValue;
  k_cells_build<<<(unsigned)strips, 1024, (size_t)cb.seen * 4, st>>>(bp, cb);
  hipError_t e = launch_cells_products(bp, cb, st);
  if (e != hipSuccess) return e;
  if (bp.act == ACT_SOFTMAX) k_cells_vjp<<<(unsigned)strips, 1024, 0, st>>>(bp, cb);
  for (int t = 0; t < 2 && e == hipSuccess; ++t)
    e = launch_mm(bp, cb, t == 1, st);
  return e;
}

}  // namespace topk
