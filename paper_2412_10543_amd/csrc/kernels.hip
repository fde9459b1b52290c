// gfx950 kernels of the RAG-synthesis attention path and their launchers:
//   prefill_varlen_kernel  packed variable-length prefill (dense K/V), several
//                          query tiles per workgroup; prefill_single_kernel: one
//   paged_decode_kernel    decode rows against a paged KV cache (split-KV
//                          partials are merged inside it by the last split
//                          of each sequence to finish)
//   mixed_kernel           decode rows and chunked-prefill pieces of a
//                          paged cache in one launch
#include <algorithm>
#include <climits>
#include <cstdlib>

#include "common.h"
#include "decode_unit.h"
#include "launch.h"
#include "prefill_tile.h"

namespace rag {

// ---------------------------------------------------------------------------
// Work order of prefill tiles.  A "stream" is one (sequence, kv head) pair;
// all q heads of its GQA group and all its query tiles read the same K/V.  A
// workgroup takes up to four of the group's q heads (a head group) and a set
// of `items` query tiles of one stream, which it runs one after another
// (prefill_items overlaps each tile's start with the end of the one before).
// The tiles of a stream are dealt to its `per` workgroups in a snake order --
// workgroup j takes tiles j, 2*per-1-j, 2*per+j, ... -- so that under the
// causal mask, where tile t costs t+1 key tiles, every workgroup of a stream
// gets nearly the same work.  Stream sigma runs on XCD sigma % 8, so every XCD
// gets the same mix of sequences (and, with 8 kv heads, exactly one kv head
// of each); on an XCD the workgroups of a stream are consecutive, so those
// resident at one time share K/V tiles through its L2.
// ---------------------------------------------------------------------------
#ifndef RAG_PF_WG_PER_CU
#define RAG_PF_WG_PER_CU 32
#endif
constexpr int kPfWgPerCu = RAG_PF_WG_PER_CU;  // workgroups per CU aimed at (load balance)
constexpr int kPfCus = 256;
constexpr int kPfMaxItems = 32;
constexpr int kBalMaxChunks = kBalMaxRows / kWave;   // balanced decode: chunks of 64 rows

struct TileCoord {
  int seq, kvh, h0, j;
  bool valid;
};

// Workgroup -> (stream, head group, workgroup j of the stream).
__device__ __forceinline__ TileCoord prefill_coord(int block, int num_streams, int hkv,
                                                   int group, int per) {
  const int hw = pf_heads_per_wg(group);
  const int ng = group / hw;
  int xcd, local;
  xcd_slot(block, xcd, local);
  const int hg = local % ng;
  const int rest = local / ng;
  TileCoord t;
  t.j = rest % per;
  const int stream = xcd + kNumXcd * (rest / per);
  t.valid = stream < num_streams;
  t.seq = stream / hkv;
  t.kvh = stream % hkv;
  t.h0 = t.kvh * group + hg * hw;
  return t;
}

// Query tile of item k of workgroup j (snake order over the per workgroups).
__device__ __forceinline__ int snake_tile(int j, int k, int per) {
  return (k & 1) ? (k + 1) * per - 1 - j : k * per + j;
}

// Items per workgroup and workgroups per (stream, head group) for a launch.
struct PfSplit {
  int items, per, n_qt;
};
// RAG_ATTN_PF_ITEMS=n (read at each launch) fixes the query tiles per
// workgroup at n instead of the load-balancing choice below: a testing and
// tuning knob (every tile is computed the same way whichever workgroup runs
// it, so outputs are bit-identical for any n).
static int pf_items_override() {
  const char* e = std::getenv("RAG_ATTN_PF_ITEMS");
  if (e == nullptr || e[0] == 0) return 0;
  const int n = std::atoi(e);
  return n >= 1 ? std::min(n, kPfMaxItems) : 0;
}

static PfSplit pf_split(int num_seqs, int hkv, int group, int max_seqlen_q, bool multi) {
  const int rows = pf_rows_per_tile(group, kPfWavesDense);
  PfSplit p;
  p.n_qt = (max_seqlen_q + rows - 1) / rows;
  const int64_t streams = (int64_t)num_seqs * hkv * (group / pf_heads_per_wg(group));
  if (!multi || p.n_qt <= 1) {
    p.items = 1;
    p.per = p.n_qt;
    return p;
  }
  if (const int forced = pf_items_override()) {
    p.items = std::min(forced, p.n_qt);
    p.per = (p.n_qt + p.items - 1) / p.items;
    return p;
  }
  const int64_t want = (int64_t)kPfWgPerCu * kPfCus;
  const int64_t per = std::max<int64_t>(1, (want + streams - 1) / std::max<int64_t>(streams, 1));
  int items = (int)std::min<int64_t>(kPfMaxItems, (p.n_qt + per - 1) / per);
  items = std::max(1, items);
  p.items = items;
  p.per = (p.n_qt + items - 1) / items;
  return p;
}

static int64_t tile_grid(int num_seqs, int hkv, int group, const PfSplit& sp) {
  const int64_t streams = (int64_t)num_seqs * hkv;
  const int64_t per_xcd = (streams + kNumXcd - 1) / kNumXcd;
  return (int64_t)kNumXcd * per_xcd * sp.per * (group / pf_heads_per_wg(group));
}

int64_t prefill_grid(int num_seqs, int hkv, int group, int max_seqlen_q) {
  return tile_grid(num_seqs, hkv, group, pf_split(num_seqs, hkv, group, max_seqlen_q, true));
}

int64_t paged_prefill_grid(int num_pieces, int hkv, int group, int max_seqlen_q) {
  return tile_grid(num_pieces, hkv, group, pf_split(num_pieces, hkv, group, max_seqlen_q, false));
}

int64_t paged_decode_grid(int num_decode, int hkv, int num_splits) {
  return (int64_t)num_decode * hkv * num_splits;
}

int64_t balanced_decode_grid(int num_decode, int hkv, int bal_units) {
  return (int64_t)hkv * (num_decode >= bal_units ? num_decode + bal_units : bal_units);
}

// Paged KV-cache write fused into the prompt prefill: the K and V rows
// [r0, r1) of one (sequence, kv head) stream go to their slots in the paged
// cache (slot = page * 16 + offset; a negative slot skips the row).  Run by
// each workgroup after its last item, for the key rows of its own query
// tiles, so every row of a sequence is written once; the rows were streamed
// through this XCD's L2 by the prefill itself.
template <int D>
__device__ __forceinline__ void prefill_rows_to_cache(const bf16_t* __restrict__ k,
                                                      const bf16_t* __restrict__ v,
                                                      size_t stride, bf16_t* __restrict__ kc,
                                                      bf16_t* __restrict__ vc,
                                                      size_t block_stride,
                                                      const int32_t* __restrict__ slots,
                                                      int r0, int r1) {
  constexpr int kCh = D / 8;
  const int n = (r1 - r0) * kCh;
  for (int p = threadIdx.x; p < n; p += 64 * kPfWavesDense) {
    const int r = r0 + p / kCh, c = p % kCh;
    const int slot = slots[r];
    if (slot < 0) continue;
    const size_t src = (size_t)r * stride + c * 8;
    const size_t dst = (size_t)(slot >> 4) * block_stride + (size_t)(slot & 15) * D + c * 8;
    const u32x4 kx = load16(k + src);
    const u32x4 vx = load16(v + src);
    *reinterpret_cast<u32x4*>(kc + dst) = kx;
    *reinterpret_cast<u32x4*>(vc + dst) = vx;
  }
}

template <int D>
__global__ __launch_bounds__(64 * kPfWavesDense, 2) void prefill_varlen_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
    const bf16_t* __restrict__ v, bf16_t* __restrict__ o, float* __restrict__ lse,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, int num_seqs,
    int hq, int hkv, int items, int per, float scale, int causal,
    bf16_t* __restrict__ k_cache, bf16_t* __restrict__ v_cache,
    const int32_t* __restrict__ slots) {
  // four K/V stages (separate arrays: the compiler then knows a DMA write to
  // one stage never aliases an LDS read of another)
  __shared__ __attribute__((aligned(16))) bf16_t st0[ChunkLayout<D>::kElemsTile];
  __shared__ __attribute__((aligned(16))) bf16_t st1[ChunkLayout<D>::kElemsTile];
  __shared__ __attribute__((aligned(16))) bf16_t st2[ChunkLayout<D>::kElemsTile];
  __shared__ __attribute__((aligned(16))) bf16_t st3[ChunkLayout<D>::kElemsTile];
  const int group = hq / hkv;
  const TileCoord tc = prefill_coord(blockIdx.x, num_seqs * hkv, hkv, group, per);
  if (!tc.valid) return;
  const int qb = cu_q[tc.seq], nq = cu_q[tc.seq + 1] - qb;
  const int kb = cu_k[tc.seq], nk = cu_k[tc.seq + 1] - kb;
  const int rows = pf_rows_per_tile(group, kPfWavesDense);
  if (tc.j * rows >= nq) return;
  const int tq = cu_q[num_seqs];
  PfGroup g;
  g.q = q + ((size_t)qb * hq + tc.h0) * D;
  g.o = o + ((size_t)qb * hq + tc.h0) * D;
  g.lse = lse ? lse + (size_t)tc.h0 * tq + qb : nullptr;
  g.q_stride = (size_t)hq * D;
  g.lse_stride = (size_t)tq;
  g.hw = pf_heads_per_wg(group);
  g.nq = nq;
  g.nk = nk;
  g.wg_rows = rows;
  g.causal = causal;
  g.scale = scale;
  DenseKV kv{k + ((size_t)kb * hkv + tc.kvh) * D, v + ((size_t)kb * hkv + tc.kvh) * D,
             (size_t)hkv * D};
  const int j = tc.j;
  prefill_items<D, kPfWavesDense, DenseKV>(
      g, kv, [j, per, rows](int it) { return snake_tile(j, it, per) * rows; }, items, st0, st1,
      st2, st3);
  // Fused cache write (prompt prefill: query rows are the key rows): the
  // first head group of the kv head writes the key rows of its query tiles.
  if (slots != nullptr && tc.h0 == tc.kvh * group) {
    const size_t block_stride = (size_t)hkv * 16 * D;
    for (int it = 0; it < items; ++it) {
      const int q0 = snake_tile(j, it, per) * rows;
      if (q0 >= nq) continue;
      prefill_rows_to_cache<D>(kv.k, kv.v, kv.stride, k_cache + (size_t)tc.kvh * 16 * D,
                               v_cache + (size_t)tc.kvh * 16 * D, block_stride, slots + kb, q0,
                               min(q0 + rows, nk));
    }
  }
}

// The same with one query tile per workgroup: no item boundaries, and the tiles
// with the most keys are dispatched first, as nothing else evens out a launch
// of few workgroups (one prompt of 3.1k tokens 106 us in ascending order, 88 so;
// 4.7k 202 -> 185, 6.2k 320 -> 301; 288 tokens of 4 heads 10.8 -> 9.8).
template <int D>
__global__ __launch_bounds__(64 * kPfWavesDense, 2) void prefill_single_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
    const bf16_t* __restrict__ v, bf16_t* __restrict__ o, float* __restrict__ lse,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, int num_seqs,
    int hq, int hkv, int n_qt, float scale, int causal, bf16_t* __restrict__ k_cache,
    bf16_t* __restrict__ v_cache, const int32_t* __restrict__ slots) {
  __shared__ __attribute__((aligned(16))) bf16_t st0[ChunkLayout<D>::kElemsTile];
  __shared__ __attribute__((aligned(16))) bf16_t st1[ChunkLayout<D>::kElemsTile];
  __shared__ __attribute__((aligned(16))) bf16_t st2[ChunkLayout<D>::kElemsTile];
  __shared__ __attribute__((aligned(16))) bf16_t st3[ChunkLayout<D>::kElemsTile];
  const int group = hq / hkv;
  const TileCoord tc = prefill_coord(blockIdx.x, num_seqs * hkv, hkv, group, n_qt);
  if (!tc.valid) return;
  const int qb = cu_q[tc.seq], nq = cu_q[tc.seq + 1] - qb;
  const int kb = cu_k[tc.seq], nk = cu_k[tc.seq + 1] - kb;
  const int rows = pf_rows_per_tile(group, kPfWavesDense);
  const int q0 = (n_qt - 1 - tc.j) * rows;
  if (q0 >= nq) return;
  const int tq = cu_q[num_seqs];
  PfGroup g;
  g.q = q + ((size_t)qb * hq + tc.h0) * D;
  g.o = o + ((size_t)qb * hq + tc.h0) * D;
  g.lse = lse ? lse + (size_t)tc.h0 * tq + qb : nullptr;
  g.q_stride = (size_t)hq * D;
  g.lse_stride = (size_t)tq;
  g.hw = pf_heads_per_wg(group);
  g.nq = nq;
  g.nk = nk;
  g.wg_rows = rows;
  g.causal = causal;
  g.scale = scale;
  const DenseKV kv{k + ((size_t)kb * hkv + tc.kvh) * D, v + ((size_t)kb * hkv + tc.kvh) * D,
                   (size_t)hkv * D};
  prefill_tile_pipe<D, kPfWavesDense, DenseKV>(g, kv, q0, st0, st1, st2, st3);
  if (slots != nullptr && tc.h0 == tc.kvh * group)
    prefill_rows_to_cache<D>(kv.k, kv.v, kv.stride, k_cache + (size_t)tc.kvh * 16 * D,
                             v_cache + (size_t)tc.kvh * 16 * D, (size_t)hkv * 16 * D, slots + kb,
                             q0, min(q0 + rows, nk));
}

// ---------------------------------------------------------------------------
// Paged kernel.  In a mixed batch the grid holds n_pf_blocks chunked-prefill
// tiles and the decode units, interleaved in groups of eight consecutive
// blocks (all tiles or all units; tile groups spread evenly through the grid)
// so that MFMA-bound tiles and HBM-bound units share the CUs instead of
// running one after the other; a tile keeps its XCD (block % 8).  Decode
// unit u is split sp = u / (num_decode * hkv) of (sequence, kv head)
// u % (num_decode * hkv), where split sp of a sequence with P pages is the
// page range [sp * pps, min((sp + 1) * pps, P)).
// ---------------------------------------------------------------------------
struct PagedKernelArgs {
  const bf16_t* q;
  const bf16_t* kc;
  const bf16_t* vc;
  bf16_t* o;
  const int32_t* tables;
  const int32_t* kv_lens;
  const int32_t* cu_q;
  float* part_o;
  float* part_lse;
  int* arrivals;              // one counter per (decode sequence, kv head)
  const bf16_t* k_new;        // appended tokens [num_decode, hkv, D] (append launch only)
  const bf16_t* v_new;
  int num_seqs, num_decode, max_blocks, hq, hkv, num_splits, pps;
  int slots;                  // partial-result slots per (row, head): workspace stride
  int bal_units;              // balanced decode: units per kv head (0: uniform splits)
  int n_pf_blocks, n_qt;
  int n_dec_groups;           // mixed batches: groups of eight decode units
  float scale;
};

// One piece of a decode row: pages [p_begin, p_end) of (row s, kv head kvh),
// split sp of n_sp, on W waves taking NP pages a step.
template <int D, int NP, int W, bool kAppend = false, bool kLoop = false>
__device__ __forceinline__ void decode_piece(const PagedKernelArgs& a, int group,
                                             size_t block_stride, int s, int kvh, int kv_len,
                                             int p_begin, int p_end, int sp, int n_sp,
                                             bf16_t* lds) {
  // decode rows come first in a batch, one query row each: row s is query row s
  const size_t head = (size_t)s * a.hq + kvh * group;
  DecodeOut out;
  out.o = a.o + head * D;
  out.part_o = a.part_o + head * a.slots * D;      // (used with more than one split only)
  out.part_lse = a.part_lse + head * a.slots;
  out.arrival = a.arrivals + (size_t)s * a.hkv + kvh;
  out.sp = sp;
  out.n_sp = n_sp;
  out.num_splits = a.slots;
  const size_t nrow = ((size_t)s * a.hkv + kvh) * D;
  decode_unit<D, NP, W, kAppend, kLoop>(
      a.q + head * D, a.kc + (size_t)kvh * 16 * D, a.vc + (size_t)kvh * 16 * D, block_stride,
      a.tables + (size_t)s * a.max_blocks, kv_len, group, p_begin, p_end, a.scale, out, lds,
      kAppend ? a.k_new + nrow : nullptr, kAppend ? a.v_new + nrow : nullptr);
}

// Decode unit u with fixed page ranges (see above), on W waves.
template <int D, int NP, int W, bool kAppend = false>
__device__ __forceinline__ void decode_block(const PagedKernelArgs& a, int u, int group,
                                             size_t block_stride, bf16_t* lds) {
  const int64_t pairs = (int64_t)a.num_decode * a.hkv;
  if ((int64_t)u >= pairs * a.num_splits) return;
  const int sp = (int)(u / pairs);
  const int pr = (int)(u % pairs);
  const int s = pr / a.hkv, kvh = pr % a.hkv;
  const int kv_len = min(a.kv_lens[s], a.max_blocks * 16);
  const int n_pages = (kv_len + 15) >> 4;
  const int n_sp = (n_pages + a.pps - 1) / a.pps;
  if (sp >= n_sp && sp > 0) return;
  const int p_begin = sp * a.pps;
  const int p_end = min(n_pages, p_begin + a.pps);
  decode_piece<D, NP, W, kAppend>(a, group, block_stride, s, kvh, kv_len, p_begin, p_end, sp,
                                  n_sp, lds);
}

// Balanced decode units: a pure decode batch is cut into units from the rows'
// actual lengths, bal_units of them per kv head where that is more than the
// rows, else at most rows + bal_units.  With as many (row, kv head) pairs as CUs
// (kFull) rows that are short or alike stay whole, one unit each (bal_skewed).
// Otherwise one of two plans, each giving row s the un consecutive units from uf
// on:
//   whole pieces   every row is cut on its own into equal pieces of at most
//                  about a quota of pages, the smallest quota tried for which
//                  the pieces fit the units: one piece per unit;
//   crossing       the pages of all rows, laid end to end, are cut into
//                  bal_units equal ranges; a unit attends the pieces of the
//                  rows its range covers, one after another.
// Crossing keeps every unit equally loaded; whole pieces spare a unit the
// second piece's chain of page-id, page and merge round trips (4-9 us on
// 20 rows of 600 tokens, whose launch is 13 us).  The plan is wave-parallel
// (one lane per row, prefix sums over the lanes; kChunks chunks of 64 rows) and
// short in code: walked row by row with integer divisions it took 3 us of that
// launch, now 0.7.
// Measured (7B heads, graph-replayed, walked and always crossing -> now): 20 rows
// x 600 tokens 20.3 -> 13.8 us, 16 x 576-1088 21.4 -> 16.6, 8 x 2.6k-10k 47.6 ->
// 43.3, 16 x 2.6k-10k 75.1 -> 72.9; 255 rows x 100-900 with one kv head 85 -> 18.

// Inclusive prefix sum over the wave's lanes.
__device__ __forceinline__ int wave_scan_add(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31
  return x;
}

// Inclusive prefix maximum of values from 0 on.
__device__ __forceinline__ int wave_scan_max(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return x;
}

// Pages (see bal_skewed).
template <int D>
constexpr float kBalOver = D == 64 ? 112.f : 56.f;
template <int D>
constexpr float kBalShort = D == 64 ? 45.f : 32.f;

// With as many (row, kv head) pairs as CUs or more: whether the rows' pages
// differ by enough for a plan to be worth it.  `over`: how many more pages the
// busiest CU has with whole rows, one workgroup each, than with an even cut.
// Fitted to 470 timed batches of 256-2000 pairs (32 to 9000 keys a row, ten head
// shapes): within 0.3% of the better of plan and whole rows on average, where
// always a plan was up to 1.4 times slower than whole rows (128 rows x 1200-1500
// keys, 2 kv heads: 33.4 us whole, 46.3 cut) and whole rows always up to 2.8
// times than a plan (32 x 100-200 keys and one of 4000, 8 kv heads: 44.0 whole,
// 15.9 cut).  40 x 2k-8k: 176 whole, 128 cut.
template <int D>
__device__ __forceinline__ bool bal_skewed(int rows, int units, int total, int longest, int group) {
  const float mean = (float)total * __builtin_amdgcn_rcpf((float)rows);
  const float even = (float)total * __builtin_amdgcn_rcpf((float)units);
  const float worst = (float)longest + mean * (float)((rows - 1) / units);
  const float over = worst - even;
  return over > kBalOver<D> * (1.f + 0.0625f * (float)group) ||
         (over > kBalShort<D> && worst > 2.f * even);
}

template <int D, int NP, int W, bool kAppend, int kChunks, bool kFull>
__device__ __forceinline__ void decode_block_balanced(const PagedKernelArgs& a, int u, int group,
                                                      size_t block_stride, bf16_t* lds,
                                                      int* keys) {
  const int kvh = u % a.hkv, k = u / a.hkv;
  const int S = a.num_decode, lane = threadIdx.x & 63, cap = a.max_blocks * 16;
  // per lane, rows 64 c + lane: keys, pages, first global page, units
  int kl[kChunks], pg[kChunks], st[kChunks], un[kChunks], uf[kChunks];
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int s = c * kWave + lane;
    kl[c] = min(a.kv_lens[min(s, S - 1)], cap);
    if (s >= S) kl[c] = 0;
  }
#pragma unroll
  for (int c = 0; c < kChunks; ++c) pg[c] = (kl[c] + 15) >> 4;
  bool uncut = false;                        // every row whole: unit k is row k
  if constexpr (kFull) {                     // (`over` is at most the longest row)
    uint64_t long_rows = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
      long_rows |= __builtin_amdgcn_ballot_w64(pg[c] > (int)kBalShort<D>);
    uncut = long_rows == 0;
  }
  int total = 0, longest = 0;
  if (!uncut) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int incl = wave_scan_add(pg[c]);
      st[c] = total + incl - pg[c];
      total += __builtin_amdgcn_readlane(incl, 63);
    }
    if constexpr (kFull) {
#pragma unroll
      for (int c = 0; c < kChunks; ++c) longest = max(longest, pg[c]);
      longest = __builtin_amdgcn_readlane(wave_scan_max(longest), 63);
      uncut = !bal_skewed<D>(S, a.bal_units, total, longest, group);
    }
  }
  if (kFull && uncut) {
    // (a second copy of the unit's code: through the plans' loop below, these
    // rows, short as a rule, took 0.4-0.7 us longer)
    if (k >= S) return;
    const int kls = min(a.kv_lens[k], cap);
    decode_piece<D, NP, W, kAppend>(a, group, block_stride, k, kvh, kls, 0, (kls + 15) >> 4, 0, 1,
                                    lds);
    return;
  }
  // Pages per unit below which the longest row could have more pieces than the
  // workspace has slots for (a crossing row also starts and ends inside one).
  float q_min = (float)kDecMinPages;
  if (a.bal_units > a.slots) {
    if constexpr (!kFull) {                  // (not the scan: 0.8% on 20 rows of 600 keys)
      longest = pg[0];
#pragma unroll
      for (int c = 1; c < kChunks; ++c) longest = max(longest, pg[c]);
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) longest = max(longest, __shfl_xor(longest, m, kWave));
      longest = __builtin_amdgcn_readfirstlane(longest);
    }
    q_min = fmaxf(q_min, (float)longest * __builtin_amdgcn_rcpf((float)(a.slots - 2)) + 2.f);
  }
  // Whole pieces: quotas from the larger of q_min and the mean per unit on, up
  // to kBalSlack pages above it.  With as many rows as units the first quota
  // fits; long rows (by their mean) are then better cut across.  (Single
  // precision: every wave of the launch computes the same numbers, and any
  // piece count up to the slots is a valid cut.)
  const bool many = S >= a.bal_units;
  const int budget = many ? S + a.bal_units : a.bal_units;
  const float q0 = fmaxf(q_min, (float)total * __builtin_amdgcn_rcpf((float)a.bal_units));
  const float q_max = many && total >= kBalLongRow * S ? 0.f : q0 + kBalSlack;
  bool whole = false;
  for (float q = q0; q <= q_max; q = fmaxf(q * 1.25f, q + 1.f)) {
    const float rq = __builtin_amdgcn_rcpf(q);
    int units = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      // (a thousandth off: a row of just the quota is one piece in spite of
      // the reciprocal's rounding)
      un[c] = pg[c] > 0 ? min(max((int)ceilf((float)pg[c] * rq - 1e-3f), 1), a.slots) : 0;
      const int incl = wave_scan_add(un[c]);
      uf[c] = units + incl - un[c];
      units += __builtin_amdgcn_readlane(incl, 63);
    }
    if (units <= budget) {
      whole = true;
      break;
    }
  }
  auto first_row = [&](auto pred) {          // first row with pred, or -1
    int s = -1;
#pragma unroll
    for (int c = kChunks - 1; c >= 0; --c) {
      const uint64_t at = __builtin_amdgcn_ballot_w64(pred(c));
      if (at != 0) s = c * kWave + __builtin_ctzll(at);
    }
    return s;
  };
  auto row = [&](const int (&v)[kChunks], int r) {
    static_assert(kChunks == 1 || kChunks == 4, "row chunk select");
    if constexpr (kChunks == 1) {
      return __builtin_amdgcn_readlane(v[0], r);
    } else {                     // (values are selected: an index would put them in memory)
      const int c = r >> 6, v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
      return __builtin_amdgcn_readlane(c == 0 ? v0 : c == 1 ? v1 : c == 2 ? v2 : v3, r & 63);
    }
  };
  int lo, hi, s;                             // this unit's global pages and first row
  uint32_t T = 0, K = 0;                     // crossing: all pages, units
  // unit holding global page g: ceil((g + 1) K / T) - 1
  auto unit_of = [&](int g) { return (int)(((uint32_t)(g + 1) * K + T - 1) / T) - 1; };
  if (whole) {
    s = first_row([&](int c) { return k < uf[c] + un[c]; });
    if (s < 0) return;
    const int n = row(un, s), sp = k - row(uf, s), p = row(pg, s);
    const float step = (float)p * __builtin_amdgcn_rcpf((float)n);
    lo = row(st, s) + (int)((float)sp * step);
    hi = row(st, s) + (sp + 1 == n ? p : (int)((float)(sp + 1) * step));
  } else {
    // at least q_min pages per unit; 32-bit arithmetic: the host takes this
    // path only when rows x table width x units stays below 2^31
    T = (uint32_t)total;
    K = max(1u, min((uint32_t)a.bal_units, (uint32_t)((float)total * __builtin_amdgcn_rcpf(q_min))));
    if ((uint32_t)k >= K) return;
    lo = (int)((uint32_t)k * T / K);
    hi = (int)((uint32_t)(k + 1) * T / K);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      uf[c] = unit_of(st[c]);
      un[c] = unit_of(st[c] + max(pg[c], 1) - 1) - uf[c] + 1;
    }
    s = first_row([&](int c) { return st[c] + pg[c] > lo; });
    if constexpr (kFull) {
      // (every wave writes the same lengths, and reads what it wrote)
#pragma unroll
      for (int c = 0; c < kChunks; ++c) keys[c * kWave + lane] = kl[c];
    }
  }
  // one call site of decode_piece: the plans' code stays one copy of the unit
  if constexpr (kFull) {
    // (what is kept per lane would sit in registers through the page loop)
    int gs = row(st, s), ps = row(pg, s), kls = row(kl, s);
    int ufs = row(uf, s), uns = row(un, s);
    for (bool first = true;; first = false) {
      if (ps > 0) {
        if (!first) __syncthreads();         // LDS of the previous piece fully read
        decode_piece<D, NP, W, kAppend, true>(a, group, block_stride, s, kvh, kls,
                                              max(lo, gs) - gs, min(hi, gs + ps) - gs, k - ufs,
                                              uns, lds);
      }
      gs += ps;
      if (++s >= S || gs >= hi) break;
      kls = __builtin_amdgcn_readfirstlane(keys[s]);
      ps = (kls + 15) >> 4;
      ufs = unit_of(gs);
      uns = unit_of(gs + max(ps, 1) - 1) - ufs + 1;
    }
  } else {
    for (bool first = true;; first = false) {
      const int gs = row(st, s), ps = row(pg, s);
      if (gs >= hi) break;
      if (ps > 0) {
        if (!first) __syncthreads();         // LDS of the previous piece fully read
        decode_piece<D, NP, W, kAppend>(a, group, block_stride, s, kvh, row(kl, s),
                                        max(lo, gs) - gs, min(hi, gs + ps) - gs, k - row(uf, s),
                                        row(un, s), lds);
      }
      if (++s >= S) break;
    }
  }
}

// Fewer (row, kv head) pairs than CUs: up to 64 rows, and up to kBalMaxRows.
template <int D, bool kAppend>
__global__ __launch_bounds__(kDecThreads, 2) void paged_decode_balanced_kernel(PagedKernelArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t lds[DecLds<D>::kBytes / 2];
  decode_block_balanced<D, kDecPages, kDecWaves, kAppend, 1, false>(
      a, blockIdx.x, a.hq / a.hkv, (size_t)a.hkv * 16 * D, lds, nullptr);
}

template <int D, bool kAppend>
__global__ __launch_bounds__(kDecThreads, 2) void paged_decode_balanced_rows_kernel(PagedKernelArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t lds[DecLds<D>::kBytes / 2];
  decode_block_balanced<D, kDecPages, kDecWaves, kAppend, kBalMaxChunks, false>(
      a, blockIdx.x, a.hq / a.hkv, (size_t)a.hkv * 16 * D, lds, nullptr);
}

// As many pairs as CUs, or more; kChunks: 1 up to 64 rows, kBalMaxChunks up to
// kBalMaxRows.  As many waves a SIMD as paged_decode_kernel, which leaves every
// row whole (with one fewer 250 rows x 100-200 keys took 39.9 us against 33.5,
// now 33.9).
template <int D, bool kAppend, int kChunks>
__global__ __launch_bounds__(kDecThreads, (D == 64 ? 3 : 2) + (kAppend ? 0 : 1)) void
paged_decode_full_kernel(PagedKernelArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t lds[DecLds<D>::kBytes / 2];
  __shared__ int keys[kChunks * kWave];
  decode_block_balanced<D, kDecPages, kDecWaves, kAppend, kChunks, true>(
      a, blockIdx.x, a.hq / a.hkv, (size_t)a.hkv * 16 * D, lds, keys);
}

// Decode rows only: one four-wave workgroup per decode unit.  kAppend: each
// row's last key is the step's new token, taken from k_new / v_new and
// stored into its cache slot by the same launch.
template <int D, bool kAppend>
__global__ __launch_bounds__(kDecThreads, 2) void paged_decode_kernel(PagedKernelArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t lds[DecLds<D>::kBytes / 2];
  decode_block<D, kDecPages, kDecWaves, kAppend>(a, blockIdx.x, a.hq / a.hkv,
                                                 (size_t)a.hkv * 16 * D, lds);
}

// Mixed batch: eight-wave workgroups.  A chunked-prefill tile runs the dense
// prefill's pipelined tile loop with K/V gathered from the paged cache; a
// decode unit runs on all eight waves (a tile workgroup fills the CU's
// registers, so a decode unit has the CU to itself and needs twice the pages
// in flight of a four-wave unit to keep its share of HBM bandwidth).
template <int D>
__global__ __launch_bounds__(64 * kPfWavesDense, 2) void mixed_kernel(PagedKernelArgs a) {
  constexpr int kE = ChunkLayout<D>::kElemsTile;
  using DL = DecLds<D, kMixedDecPages, kPfWavesDense>;
  __shared__ __attribute__((aligned(16))) bf16_t lds[4 * kE > DL::kBytes / 2 ? 4 * kE
                                                                           : DL::kBytes / 2];
  const int group = a.hq / a.hkv;
  const size_t block_stride = (size_t)a.hkv * 16 * D;
  const int64_t tile_groups = a.n_pf_blocks / kNumXcd;
  const int64_t groups = tile_groups + a.n_dec_groups;
  const int gi = blockIdx.x / kNumXcd, x = blockIdx.x % kNumXcd;
  const int tiles_before = (int)((int64_t)gi * tile_groups / groups);
  const bool is_tile = (int64_t)(gi + 1) * tile_groups / groups > tiles_before;
  if (is_tile) {
    const int num_pieces = a.num_seqs - a.num_decode;
    const TileCoord tc = prefill_coord(kNumXcd * tiles_before + x, num_pieces * a.hkv, a.hkv,
                                       group, a.n_qt);
    if (!tc.valid) return;
    const int s = a.num_decode + tc.seq;
    const int qb = a.cu_q[s], nq = a.cu_q[s + 1] - qb;
    const int rows = pf_rows_per_tile(group, kPfWavesDense);
    const int q0 = (a.n_qt - 1 - tc.j) * rows;   // tiles with the most keys first
    if (q0 >= nq) return;
    PfGroup g;
    g.q = a.q + ((size_t)qb * a.hq + tc.h0) * D;
    g.o = a.o + ((size_t)qb * a.hq + tc.h0) * D;
    g.lse = nullptr;
    g.q_stride = (size_t)a.hq * D;
    g.lse_stride = 0;
    g.hw = pf_heads_per_wg(group);
    g.nq = nq;
    g.nk = min(a.kv_lens[s], a.max_blocks * 16);
    g.wg_rows = rows;
    g.causal = 1;
    g.scale = a.scale;
    const PagedDmaKV<D> kv{a.kc + (size_t)tc.kvh * 16 * D, a.vc + (size_t)tc.kvh * 16 * D,
                           a.tables + (size_t)s * a.max_blocks, block_stride};
    prefill_tile_pipe<D, kPfWavesDense, PagedDmaKV<D>>(g, kv, q0, lds, lds + kE, lds + 2 * kE,
                                                       lds + 3 * kE);
    return;
  }
  decode_block<D, kMixedDecPages, kPfWavesDense>(a, kNumXcd * (gi - tiles_before) + x, group,
                                                 block_stride, lds);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int D>
static hipError_t launch_prefill_d(const PrefillArgs& a, hipStream_t stream) {
  const int group = a.hq / a.hkv;
  const PfSplit sp = pf_split(a.num_seqs, a.hkv, group, a.max_seqlen_q, true);
  const int64_t grid = tile_grid(a.num_seqs, a.hkv, group, sp);
  if (grid == 0) return hipSuccess;
  if (sp.items > 1)
    hipLaunchKernelGGL(prefill_varlen_kernel<D>, dim3((unsigned)grid), dim3(64 * kPfWavesDense), 0,
                       stream,
                       (const bf16_t*)a.q, (const bf16_t*)a.k, (const bf16_t*)a.v, (bf16_t*)a.o,
                       a.lse, a.cu_q, a.cu_k, a.num_seqs, a.hq, a.hkv, sp.items, sp.per, a.scale,
                       a.causal, (bf16_t*)a.k_cache, (bf16_t*)a.v_cache, a.slots);
  else
    hipLaunchKernelGGL(prefill_single_kernel<D>, dim3((unsigned)grid), dim3(64 * kPfWavesDense), 0,
                       stream,
                       (const bf16_t*)a.q, (const bf16_t*)a.k, (const bf16_t*)a.v, (bf16_t*)a.o,
                       a.lse, a.cu_q, a.cu_k, a.num_seqs, a.hq, a.hkv, sp.n_qt, a.scale, a.causal,
                       (bf16_t*)a.k_cache, (bf16_t*)a.v_cache, a.slots);
  return hipGetLastError();
}

hipError_t launch_prefill_varlen(const PrefillArgs& a, hipStream_t stream) {
  return a.d == 64 ? launch_prefill_d<64>(a, stream) : launch_prefill_d<128>(a, stream);
}

template <int D>
static hipError_t launch_paged_d(const PagedArgs& a, hipStream_t stream) {
  const int group = a.hq / a.hkv;
  PagedKernelArgs k;
  k.q = (const bf16_t*)a.q;
  k.kc = (const bf16_t*)a.k_cache;
  k.vc = (const bf16_t*)a.v_cache;
  k.o = (bf16_t*)a.o;
  k.tables = a.block_tables;
  k.kv_lens = a.kv_lens;
  k.cu_q = a.cu_q;
  k.part_o = a.part_o;
  k.part_lse = a.part_lse;
  k.arrivals = a.arrivals;
  k.k_new = (const bf16_t*)a.k_new;
  k.v_new = (const bf16_t*)a.v_new;
  k.num_seqs = a.num_seqs;
  k.num_decode = a.num_decode;
  k.max_blocks = a.max_blocks;
  k.hq = a.hq;
  k.hkv = a.hkv;
  k.num_splits = a.num_splits;
  k.pps = std::max(1, (a.max_blocks + a.num_splits - 1) / a.num_splits);
  k.slots = std::max(a.slots, a.num_splits);
  k.bal_units = a.cu_q == nullptr ? a.bal_units : 0;
  k.scale = a.scale;
  const bool mixed = a.cu_q != nullptr && a.num_seqs > a.num_decode;
  const int pf_rows = pf_rows_per_tile(group, kPfWavesDense);
  k.n_qt = mixed ? (a.max_seqlen_q + pf_rows - 1) / pf_rows : 0;
  const int64_t pf = mixed ? paged_prefill_grid(a.num_seqs - a.num_decode, a.hkv, group,
                                                a.max_seqlen_q)
                           : 0;
  k.n_pf_blocks = (int)pf;
  int64_t dec = k.bal_units > 0 ? balanced_decode_grid(a.num_decode, a.hkv, k.bal_units)
                                : paged_decode_grid(a.num_decode, a.hkv, a.num_splits);
  if (pf > 0) dec = (dec + kNumXcd - 1) / kNumXcd * kNumXcd;   // whole groups of eight
  k.n_dec_groups = (int)(dec / kNumXcd);
  const int64_t grid = pf + dec;
  if (grid > 0) {
    if (pf > 0)
      hipLaunchKernelGGL(mixed_kernel<D>, dim3((unsigned)grid), dim3(64 * kPfWavesDense), 0,
                         stream, k);
    else if (k.bal_units > 0) {
      const bool full = (int64_t)a.num_decode * a.hkv >= kDecUnits, append = a.k_new != nullptr;
      // Up to four workgroups a CU: one fewer resident than the non-appending
      // kernels' registers allow, so that the last ones go where there is room
      // (36 rows x 157-1256 keys, 16 kv heads: 42 us with two a CU, 49 with three).
      constexpr int kSpareLds = D == 128 ? 18 << 10 : 21 << 10;
      const int spare = full && !append && grid <= 4 * kDecUnits ? kSpareLds : 0;
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kDecThreads), spare, stream, k);
      };
      const bool one = a.num_decode <= kWave;
      if (full && append)
        one ? go(paged_decode_full_kernel<D, true, 1>)
            : go(paged_decode_full_kernel<D, true, kBalMaxChunks>);
      else if (full)
        one ? go(paged_decode_full_kernel<D, false, 1>)
            : go(paged_decode_full_kernel<D, false, kBalMaxChunks>);
      else if (append)
        one ? go(paged_decode_balanced_kernel<D, true>)
            : go(paged_decode_balanced_rows_kernel<D, true>);
      else
        one ? go(paged_decode_balanced_kernel<D, false>)
            : go(paged_decode_balanced_rows_kernel<D, false>);
    }
    else if (a.k_new != nullptr)
      hipLaunchKernelGGL((paged_decode_kernel<D, true>), dim3((unsigned)grid), dim3(kDecThreads),
                         0, stream, k);
    else
      hipLaunchKernelGGL((paged_decode_kernel<D, false>), dim3((unsigned)grid), dim3(kDecThreads),
                         0, stream, k);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_paged(const PagedArgs& a, hipStream_t stream) {
  return a.d == 64 ? launch_paged_d<64>(a, stream) : launch_paged_d<128>(a, stream);
}

}  // namespace rag
