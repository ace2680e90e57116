// Internal interface between the host scheduler (topk_api.hip) and the kernels
// (topk_kernels.hip). Nothing here is part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace topk {

enum Act { ACT_SOFTMAX = 0, ACT_RELU = 1 };
enum ElemType { T_F32 = 0, T_BF16 = 1 };

// Sampling modes of the fused scan: SAMPLE first estimates a per-query threshold from a
// strided subset of key tiles; THRESH takes each query's threshold from the filtered
// path's sample (PassBufs::thr).
enum ScanMode { MODE_SAMPLE = 1, MODE_THRESH = 2 };

constexpr int REDO_CAP = 1024;          // redo rows recomputed by the wide fallback kernels
constexpr int REDO_SPLIT = 512;         // keys per work item of the wide fallback
constexpr int REDO_SCORE_BLOCKS = 1024; // workgroups of the wide fallback's score kernel
constexpr int64_t FINALIZE_SLICE_BYTES = (int64_t)8 << 20;  // value matrices above this gather in column slices
constexpr int REDO_BLOCKS = 64;         // workgroups of the fallback for rows beyond REDO_CAP
constexpr int MAX_SELECT_K = 2048;  // largest k the workgroup select / finalize handle

// One call's problem. Attention: BH heads; the FFN is one head whose keys/values
// are W1/W2 (kv_head_stride = 0). Rows of Q/out are (bh * Lq + i); keys (bh, j) sit
// at K + bh * kv_head_stride + j * d.
struct Problem {
  const void* Q;
  const void* K;
  const void* V;
  void* out;
  int64_t BH, Lq, Lk, d, k, C;   // C = query chunk size; Lq = query rows per head in memory
  int64_t q0, q1;                // the rows this problem processes: [q0, q1) of every head
  int tile_only;                 // run on the chunk-tile path whatever the shape
  int64_t kv_head_stride;
  int causal;
  float scale;
  int dtype;
  int act;
  int32_t* idx_out;
  float* score_out;
};

// A pass covers chunk ids [c0, c0 + nc); chunk id = bh * nchunk + c covers query
// rows [q0 + c*C, min(q0 + (c+1)*C, q1)) of head bh. Pass-local row p = (id - c0) * C + r.
struct Pass {
  int64_t c0, nc, nchunk;
};

// Filtered chunk-tile path: every FILTER_KSTRIDE-th key is scored first; the R-th
// largest of a row's valid samples is its threshold, and the tile GEMM keeps only
// scores at or above it.
constexpr int FILTER_KSTRIDE = 16;
constexpr int64_t FILTER_MAX_LK = 65536;  // at most 4096 samples per row
// Bytes of padding after the sample buffer: the per-row threshold kernel loads up to
// 1024 samples from a row's start whatever the row's length, and discards the rest.
constexpr size_t FILTER_SAMP_PAD = 4096;

// The filtered path scores its candidates with the scan kernel (direct mode, one
// candidate list per row and half-wave) for bf16 keys of d = 128; with the MFMA tile
// GEMM (one list per row) otherwise.
inline bool filter_scan_ok(const Problem& pb) { return pb.dtype == T_BF16 && pb.d == 128; }

// Workspace pointers of one pass.
struct PassBufs {
  uint64_t* sel;      // [rows, k] selected keys, 0 pads
  int sel_sorted;     // sel in (score desc, index asc) order; 0: in the order of the candidate lists
  int32_t* redo_list; // [rows]
  int32_t* redo_count;
  float* scores;      // chunk-tile path: [rows, Lk]; fused path: redo rows [REDO_CAP + REDO_BLOCKS, Lk]
  uint64_t* cand;     // fused and filtered paths: [rows, 2, caph]
  int32_t* cnt;       // fused and filtered paths: [rows, 2]
  int64_t caph;
  int cand_single;    // one list of up to 2 caph per row, its length in cnt[2p] (fused scan,
                      // filtered tile GEMM); 0: two lists of caph, lengths cnt[2p], cnt[2p + 1]
  uint32_t* blk;      // few queries: [rows, few_row_len / 16] largest score of every 16 keys, as keys
  float* samp;        // filtered path: [rows, ceil(Lk / FILTER_KSTRIDE)] sampled scores
  float* thr;         // filtered path: [rows] thresholds
  // k_tile_scores_mfma<3>, the backward pass's products: the pairs in cell order
  const int32_t* cell_off;
  const uint32_t* cell_ent;
  const float* cell_w;
  float* cell_val;
  int64_t nstrip, ncell, off_row;
};

struct ScanCfg {
  int mode;           // ScanMode
  int stride;         // SAMPLE: one key tile in `stride` is sampled
  int R;              // SAMPLE: block maxima kept per lane, sorted (11 or 12)
  int groups;         // 32-query groups per wave (2)
  int score_only;     // the scan's score-core ablation (no filter, no candidates)
  int union_rank;     // SAMPLE: J > 0: the threshold is the J-th largest of both half-waves'
                      // lists together (13 or 20); 0: the smaller of their R-th
};

// Short rows (topk_rows.hip): calls whose rows have at most ROWS_MAX_LK keys and keep at
// most ROWS_MAX_K of them run as one kernel that needs no workspace, whatever the chunk
// size. The feature sizes are those the kernel is built for. Longer rows would not fit
// a workgroup's LDS at 32 rows each; more than 256 kept keys would need more sort scratch.
constexpr int ROWS_MAX_LK = 1024, ROWS_MAX_K = 256;
// Except for a handful of bf16 queries per head against so many keys and values that they come
// from memory: the kernel reads every value row, the general paths (few queries up to 8192
// rows, chunk tiles beyond) only the selected ones. The line lies where keys and values
// together pass 200 MB, about what the caches hold. Measured (us, this kernel / the general
// paths; in brackets before this kernel): one query per head, k = 64: 768 heads of 1024 keys, d
// 64 (201 MB) 46 / 47; 2048 heads 130 / 76 (100); 4096 heads, d 128 641 / 255 (304); of 256 keys,
// d 64 48 / 54; 512 heads of 1024, d 128, k 128 84 / 46 (72). Eight queries, 4096 heads of 1024,
// d 64 288 / 292 (457), d 128 674 / 429 (625). With more queries to share the reads this kernel
// was never the slower one than before it: sixteen, 1024 heads of 1024, d 128 196 (244).
inline bool rows_few(const Problem& pb) {
  return pb.dtype == T_BF16 && !pb.causal && pb.Lq <= 8 && pb.Lk > 256 && pb.BH * pb.Lk * pb.d * 4 > 210000000;
}
// And for d = 128 where the kernel's registers do not suffice (32 rows a workgroup, causal: its
// waves above the diagonal idle too) or the matrix instructions of few 32-bit workgroups are a
// long chain, with k <= 64: more kept keys cost the chunk tiles' select more. Measured (us, this
// kernel / chunk tiles / before this kernel): bf16, causal: 48 heads of 1024, k 8 208 / 155 / 152, k 64
// 203 / 186 / 180, k 200 200 / 316; of 600, k 64 111 / 102; 16 of 1024, k 64 81 / 78; 16 of 600 44 / 53; 96
// of 512, k 8 121 / 123. fp32: one head of 1024, k 8 40 / 30, k 64 40 / 33 (36), k 200 40 / 40; 16 rows of it
// 39 / 26 (32); two heads 40 / 37; four 41 / 55; one of 800, k 64 36 / 32; of 600 30 / 31.
inline bool rows_tiled(const Problem& pb) {
  if (pb.d != 128 || pb.k > 64) return false;
  if (pb.dtype == T_BF16) return pb.causal && pb.Lk > 512 && pb.BH * ((pb.Lq + 31) / 32) >= 512;
  return pb.Lk > 768 && pb.BH <= 2 && pb.BH * pb.Lq <= 2048;
}
// the calls the kernel can run, and those it does (the others where a given workspace is too small)
inline bool rows_can(const Problem& pb) {
  return !pb.tile_only && pb.Lk <= ROWS_MAX_LK && pb.k <= ROWS_MAX_K &&
         (pb.d == 32 || pb.d == 64 || pb.d == 96 || pb.d == 128);
}
inline bool rows_ok(const Problem& pb) { return rows_can(pb) && !rows_few(pb) && !rows_tiled(pb); }
hipError_t launch_rows(const Problem& pb, hipStream_t st);

// Few queries (k_few_scores, k_few_select): their score rows are padded to whole blocks of 16.
constexpr int64_t FEW_ROWS = 128;
__host__ __device__ inline int64_t few_row_len(int64_t Lk) { return (Lk + 15) / 16 * 16; }
hipError_t launch_few_scores(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_few_select(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
// the multi-pass select of the rows on the redo list, from score rows of row_len
hipError_t launch_tile_redo(const Problem& pb, const Pass& ps, const PassBufs& b, int64_t row_len, hipStream_t st);

hipError_t launch_init(const PassBufs& b, hipStream_t st);
hipError_t launch_tile_scores(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_tile_select(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_fused_scan(const Problem& pb, const Pass& ps, const PassBufs& b, const ScanCfg& cfg,
                             hipStream_t st);
hipError_t launch_cand_select(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_keep_select(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_redo(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_finalize(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);
hipError_t launch_mfma_probe(int32_t* rows, int32_t* cols, hipStream_t st);
hipError_t launch_mfma_rate(float* sink, uint64_t* clocks, int blocks, hipStream_t st);
// checked builds (TOPK_CHECK_INDICES): out-of-range selected indices seen by the
// finalize since the last read (the count is reset), -1 in other builds
int64_t read_bad_indices();
int mfma_rate_iters();
// Query chunking without top-k (every valid key, softmax): bf16, d in {64, 128}.
hipError_t launch_dense(const Problem& pb, const Pass& ps, hipStream_t st);

// Backward pass with input checkpointing. Rows of Q / dQ / d_out / idx / dots are
// (bh * Lq + i); keys (bh, j) of K, V, dK, dV sit at (bh * kv_head_stride + j * d)
// (the FFN is one head with kv_head_stride = 0 and X, W1, W2 as Q, K, V).
struct BwdProblem {
  const void* Q;
  const void* K;
  const void* V;
  const int32_t* idx;   // [rows, k] selected keys, entries outside [0, Lk) are padding
  const float* dots;    // [rows, k] their raw scores
  const void* dout;     // [rows, d]
  void* dQ;
  void* dK;
  void* dV;
  int64_t BH, Lq, Lk, d, k, kv_head_stride;
  float scale;
  int dtype;
  int act;
  int list_mode;  // how pairs are grouped by key, fixed for the whole call
};

// How the backward pass groups the selected pairs by key. Heads of up to 2^19 keys
// take a two-level stable bucket sort in LDS (keys in buckets of 1 << shift, at most
// BK_MAXB buckets per head, the pairs of a head in tiles of BK_TILE); the lists come
// out in increasing pair order. Larger heads count pairs with atomics on global
// counters and sort each list before summing.
constexpr int BK_TILE = 4096;
constexpr int BK_MAXB = 256;
constexpr int BK_MAXSHIFT = 11;         // at most 2048 keys per bucket
constexpr int BK_LIST_LDS = 40 * 1024;  // LDS of a list workgroup: 4 waves' counters + staged lists
struct BwdLayout {
  bool bucketed;
  int shift;        // keys per bucket = 1 << shift
  int lcap;         // list entries a bucket may stage in LDS (larger buckets write directly)
  int64_t nb;       // buckets per head
  int64_t tiles;    // tiles per head
  int64_t nhist;    // BH * nb * tiles tile counts
};
// list_mode: 0 automatic, 1 bucket sort, 2 atomic counters (as TOPK_LISTS_*)
inline BwdLayout bwd_layout(int64_t BH, int64_t Lq, int64_t Lk, int64_t k, int list_mode) {
  BwdLayout L{};
  int s = 0;
  while (((Lk + (int64_t(1) << s) - 1) >> s) > BK_MAXB) ++s;
  L.bucketed = list_mode != 2 && s <= BK_MAXSHIFT;
  L.shift = s;
  L.lcap = (BK_LIST_LDS - 4 * 4 * (1 << (s < BK_MAXSHIFT ? s : BK_MAXSHIFT))) / 4;
  L.nb = (Lk + (int64_t(1) << s) - 1) >> s;
  L.tiles = (Lq * k + BK_TILE - 1) / BK_TILE;
  L.nhist = L.bucketed ? BH * L.nb * L.tiles : 0;
  return L;
}

struct BwdBufs {
  BwdLayout L;
  float2* pair;         // [rows * k]: (activation weight, score gradient)
  int32_t* count;       // [BH * Lk + 1]: exclusive offsets of the per-key lists
  int32_t* list;        // [rows * k]: pair ids grouped by key
  int32_t* block_sums;  // scan scratch, one entry per 1024 scanned values
  int32_t* rank;        // atomic path, [rows * k]: each pair's place among its key's pairs
  uint64_t* stage;      // bucketed path, [rows * k]: pairs grouped by bucket
  int32_t* hist;        // bucketed path, [nhist + 1]: per-tile bucket counts, then offsets
};

hipError_t launch_backward(const BwdProblem& bp, const BwdBufs& b, hipStream_t st);

// Backward pass by cells of 64 rows x 64 keys (topk_cells.hip).
constexpr int CELL_MAX = 256;  // cells along a head's keys: a strip's bitmap takes 128 KB of LDS
struct CellLayout {
  int64_t nstrip, ncell;        // strips of 64 rows and cells of 64 keys per head
  int64_t off_row;              // words per strip of its ranges and its mark
  int split_q, split_k;         // parts of the d_Q products, and of the d_K and d_V products
  int64_t part_floats;          // their partial sums
};
struct CellBufs {
  int64_t nstrip, ncell, off_row;
  int seen;        // words of a strip's (row, key) bitmap
  int split_q, split_k;
  int32_t* off;    // [BH * nstrip][off_row]: each cell's range of ent
  uint32_t* ent;   // [rows * k] in cell order: local row << 6 | local key
  float* w;        // cell order: the weights
  float* a;        // cell order: d_out . V[j], then the score gradients
  float* part;     // partial sums of split products
};
CellLayout cell_layout(const BwdProblem& bp);
// d_out . V[j] of every pair into cb.a (the score GEMMs of topk_kernels.hip)
hipError_t launch_cells_products(const BwdProblem& bp, const CellBufs& cb, hipStream_t st);
hipError_t launch_backward_cells(const BwdProblem& bp, const CellBufs& cb, hipStream_t st);

// Where the products by cells take the place of the gathers by lists (bf16, automatic
// lists): where no shape that was measured is slower by more than the runs differ. The gathers'
// time goes with the pairs and the row size (0.8 ps per pair and feature), and with few rows
// with k (about 0.8 us a kept key); the products' with rows x keys (6 ps at d = 256, 15 to 18 at
// 768 to 1024) and, in few workgroups, with the longest walk along a head's cells.
// The causal mask, which the backward pass is not told of, leaves the gathers their time and
// makes those walks uneven. Measured (us, lists / cells; c: causal):
//  d = 64: 32 heads of 1024, k 64 176 / 148, c 175 / 184; 40 of 1000, 63 209 / 213; 48 of 1024, 64
//   247 / 215, c 248 / 238; 43 of 768, 48 168 / 169, c 173 / 141; 64 of 512, 32 171 / 94, c 173 / 107;
//   longer heads 24 of 1500, 94 217 / 293; 12 of 2048, 128 189 / 238.
//  d = 128, one key in 16: 32 heads of 512 117 / 88, c 120 / 96; of 1024: 16 138 / 120, c 139 / 153; 24
//   187 / 162, c 191 / 201; 32 236 / 169, c 236 / 212; of 2048: 16 359 / 301, c 355 / 378; 24 535 / 474, c
//   534 / 474; one in 12: 16 of 2048 471 / 333, c 465 / 431; one in 32: 16 of 4096 726 / 902; k 512: 2 of
//   8192 779 / 667, c 1063 / 910. d = 160: 16 of 1024, 64 205 / 150, c 207 / 178.
//  d = 256: 16 heads of 1024, k 64 203 / 160, c 208 / 188; 8 of them 129 / 125, c 135 / 145; one key in
//   24: 8 of 2048 249 / 246, c 247 / 283; 24 664 / 617, c 666 / 571; k 256: 1 head of 4096 221 / 200, c 340
//   / 295; one in 32: heads of 512: 16 78 / 87, 32 117 / 106, c 120 / 106; 32 of 1024 233 / 209, c 237 / 223; 64
//   of 100, k 4 68 / 50; of
//   2048: 24 504 / 573, 64 1371 / 1330, c 1392 / 1122. d = 768, one in 32: 16 of 512 125 / 128, 32 212 / 171; 32
//   of 1024 605 / 504; 24 of 2048 1743 / 1403, c 1605 / 1113; 512 heads of one row and 1000 keys 787 / 1023.
//  Feed-forward d = 256: 4096 tokens and units: k 256 221 / 189, 170 161 / 170; 512 tokens, 1024, 64 60
//   / 73; 8192, 1024, 64 187 / 146; 8192, 4096, 170 280 / 274; 8192, 8192, 256 422 / 478; 8192, 16384, 512
//   922 / 802.
//  d >= 512 (tokens, d, units, k): 512, 512, 1024, 64 89 / 82; 512, 768, 768, 32 72 / 83; 2048, 768, 300, 20
//   130 / 97; 2048, 512, 4096, 170 210 / 170; 4096, 1024, 2048, 85 247 / 260; 4096, 512, 4096, 128 218 / 257;
//   16384 of these 800 / 768; 128 of these 131 / 87; 4096, 768, 4096, 128 355 / 339, k 100 295 / 335; 2048, 1024,
//   8192, 256 468 / 394; 2048, 768, 16384, 410 688 / 580; 8192, 768, 8192, 200 1103 / 1177; 16384 of these
//   2365 / 2270; 16384, 768, 4096, 512 5263 / 1445; 64, 1024, 2048, 64 86 / 76; 1, 768, 4096, 512 402 / 79.
// cells_can: the calls that can run by cells (also where a given workspace does not hold the lists).
inline bool cells_can(const BwdProblem& bp) {
  if (bp.list_mode != 0 || bp.dtype != T_BF16 || bp.d % 32 != 0 || bp.Lk > (int64_t)64 * CELL_MAX) return false;
  // every launch below 2^32 threads: 1024 a strip; 256 a tile of the products, whose column
  // tiles (at most four) and two sides make eight at most
  const int64_t tq = (bp.Lq + 127) / 128, tk = (bp.Lk + 127) / 128;
  if (bp.BH * ((bp.Lq + 63) / 64) >= 1 << 22 || bp.BH * (tq > tk ? tq : tk) * 8 >= 1 << 24 || bp.BH * tq * tk >= 1 << 24) return false;
  return bp.d == 64 || bp.d >= 128;
}
inline bool cells_ok(const BwdProblem& bp) {
  if (!cells_can(bp)) return false;
  const int64_t d = bp.d, k = bp.k, Lk = bp.Lk, tiles = bp.BH * ((bp.Lq + 127) / 128);
  if (d == 64) return Lk <= 16 * k && Lk <= 1024 && tiles >= (Lk <= 768 ? 256 : 384);
  if (d < 256) {
    if (Lk > 16 * k) return false;
    return (k >= 512 && tiles >= 64) || tiles >= (d > 128 || Lk <= 512 ? 128 : Lk <= 1024 || Lk <= 12 * k ? 256 : 384);
  }
  int64_t most = 0;  // keys or units per kept one
  if (bp.act == ACT_SOFTMAX) {
    if (d >= 512 && Lk > 512 && bp.Lq < 64 && k < 128) return false;
    if (tiles >= 128 || (k >= 256 && tiles >= 16)) most = 16;
    if (tiles >= 384) most = 25;
    if (tiles >= 64 && Lk <= 320) most = 32;
    if (tiles >= (Lk <= 512 ? 128 : Lk <= 1024 ? 256 : d >= 512 ? 384 : 1024)) most = Lk <= 512 ? 40 : 34;
    return Lk <= most * k;
  }
  const int64_t N = bp.Lq;
  if (d >= 512) {
    if (k >= 64 || N >= 2048) most = 16;
    if (k >= 128 || N >= 8192) most = 25;
    if (k >= 256 || (k >= 128 && d >= 768) || (k >= 64 && N <= 128) || N >= 16384) most = 32;
    if (k >= 400 || (k >= 200 && N >= 16384)) most = 40;
  } else {
    if (k >= 128 || N >= 8192) most = N >= 8192 ? 25 : 16;
    if (k >= 512 && N >= 8192) most = 32;
  }
  return Lk <= most * k;
}
hipError_t launch_filter(const Problem& pb, const Pass& ps, const PassBufs& b, int stage, hipStream_t st);
hipError_t launch_filter_scan(const Problem& pb, const Pass& ps, const PassBufs& b, hipStream_t st);

}  // namespace topk
