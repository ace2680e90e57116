// Query chunking with the top-k disabled: the paper's comparison baseline
// (Section 2.2, "Query chunking"; Section 3 compares top-k attention against it).
// Every valid key of a query contributes: out_i = sum_j softmax_j(scale * q_i.k_j) v_j
// (Eq. 1, with the causal mask of Eq. 2), the k = Lk fixed point of Eq. 4.
//
// gfx950 kernel, bf16 inputs, fp32 accumulation, d in {64, 128}: a streaming softmax
// over key tiles, so no [C, Lk] score tile is ever written. One workgroup = 4 waves x 32
// queries of one query chunk of one head. Per 64-key tile:
//   * scores S^T = K Q^T by v_mfma_f32_32x32x16_bf16 (K tile from LDS as the A
//     operand, the wave's 32 queries in registers as B): lane l holds 16 keys'
//     scores of query l % 32 per 32-key block, keys 8*(v/4) + 4*(l/32) + v%4;
//   * the running row maximum and sum are per query (the two lanes of a query,
//     l and l + 32, exchange their maxima); the accumulator is rescaled in tiles where some
//     query's maximum grows;
//   * O^T += V^T P^T by the same MFMA: the B operand is the lane's own 8 softmax
//     weights of a 16-key step, in the order the score layout holds them, and the
//     A operand holds V^T in that same key order: column n * D/32 + c of V is row n of
//     feature block c, so a lane reads D/32 neighbouring columns of 8 rows of the V tile
//     (which stays as it is in memory) and pairs them up by byte permutes.
// K and V tiles come by direct global-to-LDS loads, one tile ahead.
//
// Bound by vector instructions: per tile and wave 32 exponentials (512 cycles) and about
// 160 others (640) beside 16 MFMAs (512), which this chip overlaps only in part (1670
// cycles measured). Against V transposed through registers with 2-byte LDS writes, the
// library exp2f and a rescale in every tile: 12 heads of 8192 tokens, d = 64: 424 -> 284 us.
// The exponential instruction alone makes a weight below 2^-126 zero; a tile whose lowest
// score leads there adds those weights by themselves (the test for it takes 14 of 284 us).
// (Taking a new maximum over only once it exceeds the old by 2^8 in weight ran 290 us, but
// the largest weight is then not exactly 1 and its rounding shows: 2.34e-3 against 2.28e-3.)
#include "topk_internal.h"

#include <math.h>

#include <type_traits>

namespace topk {

typedef __bf16 dbf16x8 __attribute__((__vector_size__(16)));
typedef __bf16 dbf16x4 __attribute__((__vector_size__(8)));
typedef float df32x16 __attribute__((__vector_size__(64)));

// s_waitcnt immediate: no vector-memory operation outstanding, the other counters ignored
constexpr int DENSE_WAIT_VM0 = (7 << 4) | (15 << 8);

constexpr int DN_KT = 64;   // keys per tile
constexpr int DN_QW = 32;   // queries per wave
constexpr int DN_QB = 4 * DN_QW;

struct DenseArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  uint16_t* out;
  int64_t Lq, Lk, C, kv_head_stride;  // Lq: query rows per head in memory
  int64_t c0, nchunk, wgs_per_chunk;
  float scale_log2e;                  // scale * log2(e)
};

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void k_dense_attn(DenseArgs a) {
  constexpr int NS = D / 16;         // MFMA steps over the features (scores)
  constexpr int CH = 2 * D / 16;     // 16-byte parts per key row
  constexpr int TILEB = DN_KT * 2 * D;
  constexpr int LPW = TILEB / 1024 / 4;
  constexpr int NDB = D / 32;        // 32-row blocks of the output features
  constexpr int VW = NDB / 2;        // words of a lane's columns of a V row
  __shared__ __attribute__((aligned(16))) unsigned char ks0[TILEB];
  __shared__ __attribute__((aligned(16))) unsigned char ks1[TILEB];
  __shared__ __attribute__((aligned(16))) unsigned char vs0[TILEB];
  __shared__ __attribute__((aligned(16))) unsigned char vs1[TILEB];

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5,
            n = lane & 31;
  const int64_t NG = gridDim.x, bid = blockIdx.x;
  int64_t wg = (NG % 8 == 0) ? (bid % 8) * (NG / 8) + bid / 8 : bid;
  if (CAUSAL) wg = NG - 1 - wg;  // the longest workgroups first
  const int64_t cl = wg / a.wgs_per_chunk, blk = wg - cl * a.wgs_per_chunk;
  const int64_t id = a.c0 + cl, bh = id / a.nchunk, c = id - bh * a.nchunk;
  const uint16_t* Kh = a.K + bh * a.kv_head_stride;
  const uint16_t* Vh = a.V + bh * a.kv_head_stride;
  const int64_t q_first = c * a.C + blk * DN_QB;
  int64_t q_last = c * a.C + (blk * DN_QB + DN_QB < a.C ? blk * DN_QB + DN_QB : a.C) - 1;
  q_last = q_last < a.Lq - 1 ? q_last : a.Lq - 1;
  const int64_t ntiles_all = (a.Lk + DN_KT - 1) / DN_KT;
  const int64_t ntiles = CAUSAL && q_last / DN_KT + 1 < ntiles_all ? q_last / DN_KT + 1 : ntiles_all;

  const int64_t local = blk * DN_QB + wave * DN_QW + n;  // the lane's query within the chunk
  const int64_t qi = c * a.C + local;                      // its index within the head
  const bool ok = local < a.C && qi < a.Lq;
  dbf16x8 b[NS];
  {
    const uint16_t* q = a.Q + (bh * a.Lq + (ok ? qi : 0)) * D + (D / 2) * half;
#pragma unroll
    for (int s = 0; s < NS; ++s) b[s] = ok ? *(const dbf16x8*)(q + 8 * s) : (dbf16x8){};
  }

  // tile t of K (16-byte parts XOR-swizzled by row, as in the fused scan) and of V (as it
  // lies in memory); rows past Lk load the last key, their scores are masked
  auto issue = [&](int64_t t, unsigned char* kd, unsigned char* vd) {
    const int left = (int)(a.Lk - t * DN_KT < DN_KT ? a.Lk - t * DN_KT : DN_KT) - 1;
    const uint16_t* kt = Kh + t * DN_KT * D;
    const uint16_t* vt = Vh + t * DN_KT * D;
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      const int cidx = (wave * LPW + j) * 64 + lane, r = cidx / CH, rr = min(r, left);
      __builtin_amdgcn_global_load_lds((const void*)(kt + (uint32_t)(rr * D + ((cidx % CH) ^ (r & 7)) * 8)),
                                       (__attribute__((address_space(3))) void*)&kd[(wave * LPW + j) * 1024], 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)(vt + (uint32_t)(rr * D + (cidx % CH) * 8)),
                                       (__attribute__((address_space(3))) void*)&vd[(wave * LPW + j) * 1024], 16, 0, 0);
    }
  };

  df32x16 o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) o[db] = (df32x16){};
  float m_run = -INFINITY, l_run = 0.f;
  const float cexp = a.scale_log2e;

  // scores of the 32-key block rb of the tile for the lane's query
  auto block_scores = [&](const unsigned char* kb, int rb) {
    const int r = rb * 32 + n;
    dbf16x8 av[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) av[s] = *(const dbf16x8*)(kb + (r * CH + ((half * NS + s) ^ (r & 7))) * 16);
    df32x16 acc = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[s], b[s], acc, 0, 0, 0);
    return acc;
  };
  auto mask = [&](df32x16& acc, int64_t jb) {  // jb: key of register 0 of this lane
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t j = jb + 8 * (v >> 2) + (v & 3);
      if (j >= a.Lk || (CAUSAL && j > qi)) acc[v] = -INFINITY;
    }
  };
  auto tile = [&](int64_t t, const unsigned char* kb, const unsigned char* vb) {
    df32x16 s[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) s[rb] = block_scores(kb, rb);
    // the tile's lowest score (masked keys' included: they only choose the exponential below)
    float low = INFINITY;
#pragma unroll
    for (int v = 0; v < 32; v += 2)
      low = __builtin_elementwise_minimum(__builtin_elementwise_minimum(low, s[v >> 4][v & 15]), s[v >> 4][(v & 15) + 1]);
    if (t * DN_KT + DN_KT > a.Lk || (CAUSAL && t * DN_KT + DN_KT - 1 > q_first + wave * DN_QW)) {
      mask(s[0], t * DN_KT + 4 * half);
      mask(s[1], t * DN_KT + 32 + 4 * half);
    }
    // the tile's maximum of the query (both of its lanes)
    float mt = -INFINITY;
#pragma unroll
    for (int v = 0; v < 32; v += 2)
      mt = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mt, s[v >> 4][v & 15]), s[v >> 4][(v & 15) + 1]);
    mt = __builtin_elementwise_maximum(mt, __shfl_xor(mt, 32, 64));
    // (not <=: for NaN too; queries whose maximum stays multiply by 1)
    if (__builtin_amdgcn_ballot_w64(!(mt <= m_run))) {
      const float m_new = fmaxf(m_run, mt);
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((m_run - m_new) * cexp);  // m_run = -inf -> 0
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
    }
    const float off = m_run == -INFINITY ? 0.f : m_run * cexp;  // all keys masked so far: weights stay 0
    auto values = [&](auto tiny) {
      int at = 4 * half * 2 * D + n * NDB * 2;  // the lane's place in V's tile
      float bias = -off;
      if (decltype(tiny)::value) asm volatile("" : "+v"(at), "+v"(bias));  // (nothing of one pass is held for the other)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          if (decltype(tiny)::value) __builtin_amdgcn_sched_barrier(0);  // one step's registers at a time
          // B: the lane's 8 weights of keys 16 st + {4h..4h+3, 8+4h..8+4h+3} of the block
          dbf16x8 pb;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = fmaf(s[rb][8 * st + e], cexp, bias);
            const float w = !decltype(tiny)::value ? __builtin_amdgcn_exp2f(x) : x < -126.f ? exp2f(x) : 0.f;
            l_run += w;
            pb[e] = (__bf16)w;
          }
          // A: rows 32 rb + 16 st + the same keys of V, columns n * NDB ..
          uint32_t vr[8][VW];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int key = rb * 32 + 16 * st + (e & 4) * 2 + (e & 3);
            __builtin_memcpy(vr[e], __builtin_assume_aligned(vb + at + key * 2 * D, 4 * VW), 4 * VW);
          }
#pragma unroll
          for (int db = 0; db < NDB; ++db) {
            const uint32_t sel = db & 1 ? 0x07060302u : 0x05040100u;
            const int w = db / 2;
            const uint4 av = make_uint4(__builtin_amdgcn_perm(vr[1][w], vr[0][w], sel), __builtin_amdgcn_perm(vr[3][w], vr[2][w], sel),
                                        __builtin_amdgcn_perm(vr[5][w], vr[4][w], sel), __builtin_amdgcn_perm(vr[7][w], vr[6][w], sel));
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(dbf16x8, av), pb, o[db], 0, 0, 0);
          }
        }
      }
    };
    // weights below the smallest normal number, which the exponential instruction alone makes
    // 0, are added by themselves where the tile has any
    if (__builtin_amdgcn_ballot_w64(fmaf(low, cexp, -off) < -126.f)) {
      values(std::true_type{});
    }
    values(std::false_type{});
  };

  // One tile of lookahead: before tile t is read, this wave's loads of it are complete and
  // the barrier publishes every wave's part; it also proves that no wave still reads the
  // buffers the next loads overwrite. The buffers are named at compile time, so that reads
  // of one pair do not wait for the loads into the other.
  if (ntiles > 0) issue(0, ks0, vs0);
  for (int64_t t = 0; t < ntiles; t += 2) {
    __builtin_amdgcn_s_waitcnt(DENSE_WAIT_VM0);
    __syncthreads();
    if (t + 1 < ntiles) issue(t + 1, ks1, vs1);
    tile(t, ks0, vs0);
    if (t + 1 >= ntiles) break;
    __builtin_amdgcn_s_waitcnt(DENSE_WAIT_VM0);
    __syncthreads();
    if (t + 2 < ntiles) issue(t + 2, ks0, vs0);
    tile(t + 1, ks1, vs1);
  }
  if (!ok) return;
  const float l = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = l > 0.f ? 1.f / l : 0.f;
  uint16_t* dst = a.out + (bh * a.Lq + qi) * D;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    // rows 8 g + 4 h .. + 3 of every block: features (8 g + 4 h) * NDB .. of the lane's query
    dbf16x4 w[NDB];
#pragma unroll
    for (int e = 0; e < 4 * NDB; ++e) w[e / 4][e % 4] = (__bf16)(o[e % NDB][4 * g + e / NDB] * inv);
#pragma unroll
    for (int q = 0; q < NDB; ++q) *(dbf16x4*)(dst + (8 * g + 4 * half) * NDB + 4 * q) = w[q];
  }
}

hipError_t launch_dense(const Problem& pb, const Pass& ps, hipStream_t st) {
  DenseArgs a;
  a.Q = (const uint16_t*)pb.Q;
  a.K = (const uint16_t*)pb.K;
  a.V = (const uint16_t*)pb.V;
  a.out = (uint16_t*)pb.out;
  a.Lq = pb.Lq;
  a.Lk = pb.Lk;
  a.C = pb.C;
  a.kv_head_stride = pb.kv_head_stride;
  a.c0 = ps.c0;
  a.nchunk = ps.nchunk;
  a.wgs_per_chunk = (pb.C + DN_QB - 1) / DN_QB;
  a.scale_log2e = pb.scale * 1.4426950408889634f;
  const int64_t g = ps.nc * a.wgs_per_chunk;
  if (g > 0x7FFFFFFF) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)g;
  if (pb.d == 64 && !pb.causal) k_dense_attn<64, false><<<grid, 256, 0, st>>>(a);
  else if (pb.d == 64) k_dense_attn<64, true><<<grid, 256, 0, st>>>(a);
  else if (pb.d == 128 && !pb.causal) k_dense_attn<128, false><<<grid, 256, 0, st>>>(a);
  else if (pb.d == 128) k_dense_attn<128, true><<<grid, 256, 0, st>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace topk
