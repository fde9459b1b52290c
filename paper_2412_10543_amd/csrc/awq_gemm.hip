// Group-quantized int4-weight x bf16-activation GEMM for gfx950: Y = X W with
// W[k, n] = (q[k, n] - z[g, n]) * s[g, n], g = k / 128 (the AWQ weight format
// of the served models, Sec. "Setup").
//
// Method.  The 4-bit codes become MFMA operands without any floating-point
// dequantization: a code q placed in the low mantissa bits of the bf16 value
// 128.0 (bits 0x4300 | q) is exactly 128 + q, so two codes become a pair of
// bf16 operands with one shift and one and-or.  For group g,
//     sum_k X[m, k] W[k, n] = s[g, n] * (P[m, n] - (128 + z[g, n]) * S[g, m]),
//     P = sum_k X[m, k] (128 + q[k, n]),   S[g, m] = sum of X[m, k] over g.
// Larger batches (awq_gemm_md_kernel): S, formed by the kernel beside its
// products, is stored as three bf16 pieces S1 + S2 + S3 = S (exact: 24 bits in
// 3 x 8), and the zero-point term becomes one more MFMA per group (A = the
// pieces, B = -(128 + z), which bf16 holds exactly as bits 0xC300 | z), with a
// running rescale of the accumulators for the scale (see there).  Small
// batches (awq_gemm_sm_kernel): the kernel stages its slice of X in LDS, forms
// S with the matrix cores (X times a ones operand), then applies zero point
// and scale with two fp32 FMAs per output element and group.
//
// Packed weight layout (rag_awq_pack_weights): int32 [K/128][N][16].  The
// 16 words of (group g, column n) are 64 contiguous bytes; word
// 8a + 4b + c holds the codes of the k-octet o = 4c + 2b + a, i.e. of
// k = 128g + 8o + j, j = 0..7, code j in bits 4(j/2) + 16(j%2) .. +4.  This
// order serves both MFMA shapes with contiguous reads: a 32x32x16 B-operand
// lane (column, half h) needs the octets 2t + h of k-steps t = 0..7, which
// are words 8h .. 8h+7 (step t at 8h + 4(t&1) + t/2); a 16x16x32 lane
// (column, quarter qq) needs the octets 4t + qq of k-steps t = 0..3, words
// 8(qq&1) + 4(qq>>1) .. +3.
#include <cstdint>
#include <cstdlib>

#include "common.h"
#include "awq.h"

namespace rag {

constexpr int kAwqGroup = 128;
constexpr int kAwqCus = 256;     // MI355X compute units

// A value the compiler must keep in a VGPR (no constant folding).
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Four bf16 pairs (128 + code) from one packed word.  mask = 0x000F000F and
// magic = 0x43004300 come in registers: gfx9 VOP3 instructions take no
// literal operand, and with both constants in VGPRs each pair is one
// v_and_or_b32 (after a shift).
__device__ __forceinline__ bf16x8 codes_to_bf16(uint32_t w, uint32_t mask, uint32_t magic) {
  u32x4 r;
  r[0] = (w & mask) | magic;
  r[1] = ((w >> 4) & mask) | magic;
  r[2] = ((w >> 8) & mask) | magic;
  r[3] = ((w >> 12) & mask) | magic;
  return as_bf16x8(r);
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) {
  return __builtin_bit_cast(float, bits16 << 16);
}

// vmcnt <= n (n < 64), expcnt and lgkmcnt unconstrained.
template <int n>
__device__ __forceinline__ void wait_vm() {
  static_assert(n >= 0 && n < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (n & 15) | ((n >> 4) << 14));
}

// Per-column constants of one group from its bf16 scale bits: c = sign * m, the
// conversion mask and magic (exponent field 134 + e), and the bf16 bits of
// -(128 + z) 2^e.  Scales of 2^41 and above keep the excess power of two in c:
// (128 + q) 2^e x is summed before the zero point cancels most of it, and no
// scale may take that sum out of range that leaves the result in it.
struct ColScale {
  float c;
  uint32_t mask, magic, nz;
};
constexpr uint32_t kMaxOperandExp = 127 + 40;
// Normal scales (plain_scale): 13 instructions.
__device__ __forceinline__ bool plain_scale(uint32_t sb) {
  const uint32_t E = sb & 0x7F80u;
  return E - 0x80u < 0x7F80u - 0x80u;
}
__device__ __forceinline__ ColScale col_scale_plain(uint32_t sb, uint32_t z) {
  const uint32_t field = min(sb & 0x7F80u, kMaxOperandExp << 7);
  const uint32_t ex = field + (7u << 7);                // exponent field 134 + e
  ColScale r;
  r.c = bf16_to_f32(sb - field + 0x3F80u);
  r.mask = 0x000F000Fu;
  r.magic = ex | (ex << 16);
  r.nz = 0x8000u | ex | z;
  return r;
}
// The others.  A zero scale gives mask = magic = nz = 0 and c = 0 (the caller
// keeps its reference).  Infinity gives c = infinity: the caller's u, y / c, drops
// what it held (0 where that was finite) and takes the group's own sum, which
// times c is infinity of its sign, or NaN where it is 0, as y + inf * sum is.  (A
// second infinite scale in a column of one workgroup's groups gives NaN.)
__device__ __forceinline__ ColScale col_scale(uint32_t sb, uint32_t z) {
  if (plain_scale(sb)) return col_scale_plain(sb, z);
  const uint32_t mt = sb & 0x7Fu;
  const int k = 31 - __builtin_clz(mt | 1u);            // subnormal: mt * 2^-133
  const bool subnormal = (sb & 0x7F80u) == 0, zero = subnormal && mt == 0;
  const uint32_t ex = (uint32_t)(134 + (subnormal ? k - 133 : 0)) << 7;
  const float m = bf16_to_f32((sb & 0x8000u) | 0x3F80u | ((mt << (7 - k)) & 0x7Fu));
  ColScale r;
  r.c = zero ? 0.f : subnormal ? m : bf16_to_f32(sb);   // (infinity or NaN as it is)
  r.mask = zero ? 0u : 0x000F000Fu;
  r.magic = zero ? 0u : ex | (ex << 16);
  r.nz = zero ? 0u : 0x8000u | ex | z;
  return r;
}

// ---------------------------------------------------------------------------
// Larger batches: workgroups of NW waves own 32 MB x 64 NW tiles of Y; wave w
// computes all rows and the columns 64 w .. +64 as MB x 2 MFMA blocks of 32 x 32.
// The X tile of a group is shared through LDS (direct global -> LDS copies one
// group ahead, two stages; row r's 16-byte chunk c at position c ^ (r & 15), so
// that the A reads of 16 rows hit 16 distinct bank groups); the code words, scales
// and zero points belong to one wave only and go from memory straight into its
// registers, one group ahead.
//
// Group sums.  Each wave sums its share of the rows of the X tile (one lane per
// row and half of a k-step, v_dot2 with ones) and stores the sums as three
// bf16 pieces (exact) in LDS in the A layout; the zero-point MFMA of a group is
// issued after the next barrier, when every wave's pieces are visible.
//
// Scale handling.  Each scale is split exactly as s = m * 2^e with |m| in
// [1, 2).  The power of two goes into the B operands: the magic constant's
// exponent field becomes 134 + e, so a code turns into (128 + q) 2^e, still
// exact in bf16 (likewise -(128 + z) 2^e for the zero-point term).  The
// accumulators hold u = y / c with c the m of the column's last group: before
// group g they are multiplied by c / m[g, n] (one fp32 multiply per element;
// the ratio lies in (1/2, 2), so u never leaves the range of y), then every
// MFMA of group g accumulates straight into them, and y = u * c at the end.  A
// zero scale turns the column's operands to zero (mask and magic 0) and leaves
// c as it was.
//
// What bounds it.  The matrix cores with 128-row tiles (hardware counters: busy
// 64-70% of the cycles at 8192 rows, 38% with gate_up's 160-row tiles at 320: 72
// MFMAs a wave and group beside 340 vector instructions, 44 LDS reads);
// vector issue with the low tiles, where a converted code word serves fewer row
// blocks; round trips (first loads, split merge) on small grids.  So each k-step
// issues one MFMA, then a share of the next step's conversions, LDS reads,
// copies and sums, and the rescale of a block runs under the first two k-steps
// of the block before it: left to the compiler, 180 vector instructions in a
// row kept the matrix cores idle each group (gate_up, 320 rows, 160-row tile:
// 98 us against 87 now; 8192 rows, 128 x 256: 1804 against 1684).
// Tiles.  Four waves, two workgroups a CU, whose barriers then do not stall
// both; eight waves where 128 x 512 tiles fill the chip (half the X copies:
// 8192 rows 353 / 233 / 1632 / 809 us for qkv / o / gate_up / down against 366 /
// 246 / 1697 / 850 with four).  The kernels replaced (group-sum pass, 128 x 512
// tiles split 3 to 19 ways with a reduce pass on small grids): 372 / 252 / 1654
// / 853 us at 8192 rows, 60 / 53 / 135 / 84 at 320 rows against 29 / 23 / 87 / 53.
// ---------------------------------------------------------------------------
namespace awq_md {
constexpr int kGroupM = 8;                       // M tiles per raster group
constexpr int kOutStride = 144;                  // bytes per row of the output transpose
constexpr int kMaxSplitTiles = 320;              // (more tiles fill the chip unsplit)
template <int MB, int NW>
struct Shape {
  static constexpr int kBM = 32 * MB;
  static constexpr int kBN = 64 * NW;
  static constexpr int kX = kBM * kAwqGroup * 2;           // one stage
  static constexpr int kSP = kBM * 32;                     // pieces: [row][half][2 parts x 4]
  static constexpr int kLds = 2 * kX + 2 * kSP;
  // Group sums are formed in 2 MB units of (32 rows, 4 of the 8 k-steps), unit
  // w + NW i by wave w.
  static constexpr int kUnits = 2 * MB;
  static constexpr int kPer = (kUnits + NW - 1) / NW;
  static constexpr int kCopies = 8 * MB / NW;              // X copy instructions per wave
  static_assert(NW * 32 * kOutStride <= kLds, "output transpose fits");
};
}  // namespace awq_md

__device__ __forceinline__ float dot2_ones(uint32_t pair, float acc) {
  const uint32_t one = 0x3F803F80u;
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair),
                                         __builtin_bit_cast(bf16x2, one), acc, false);
}

template <int MB, int NW, bool kSplit>
__global__ __launch_bounds__(64 * NW, MB == 1 ? 3 : MB > 4 ? 1 : 2) void
awq_gemm_md_kernel(const bf16_t* __restrict__ x, const uint32_t* __restrict__ qw,
                   const bf16_t* __restrict__ scales, const uint8_t* __restrict__ zeros,
                   bf16_t* __restrict__ y, float* __restrict__ part, int* __restrict__ arrivals,
                   int M, int N, int K, int groups_per_split, int splits, int tiles_m,
                   int tiles_n, int tiles_per_xcd) {
  using namespace awq_md;
  using Sh = Shape<MB, NW>;
  __shared__ __attribute__((aligned(16))) char lds[Sh::kLds];
  const int lane = threadIdx.x & 63, w = wave_id();
  const int r = lane & 31, h = lane >> 5;
  // tile: XCD-contiguous ranges of a grouped raster order (kGroupM M-tiles per
  // group, M fastest within it), so the workgroups resident on one XCD share X
  // rows and code columns in its L2
  int xcd, local;
  xcd_slot(blockIdx.x, xcd, local);
  const int pid = xcd * tiles_per_xcd + local;
  if (local >= tiles_per_xcd || pid >= tiles_m * tiles_n) return;
  const int per_group = kGroupM * tiles_n;
  const int first_m = (pid / per_group) * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int mt = first_m + (pid % per_group) % gm;
  const int nt = (pid % per_group) / gm;
  // the last row tile ends at row M - 1 (the host picks 32 MB <= M, or MB = 1):
  // the rows it shares with the tile before are computed twice, to the same bits
  const int m0 = max(0, min(mt * Sh::kBM, M - Sh::kBM)), n0 = nt * Sh::kBN + 64 * w;
  const int groups = K / kAwqGroup;
  const int g_begin = blockIdx.y * groups_per_split;
  const int n_groups = min(groups, g_begin + groups_per_split) - g_begin;
  const bool cols_in = n0 < N;                   // N is a multiple of 128: whole waves

  // ---- per-lane byte offsets, the same for every group: copy j moves rows
  // 4 (kCopies w + j) + lane / 16, so copies four apart differ by 16 rows ----
  constexpr int kOffs = Sh::kCopies < 4 ? Sh::kCopies : 4;
  uint32_t xoff[kOffs];
#pragma unroll
  for (int j = 0; j < kOffs; ++j) {
    const int row = 4 * (Sh::kCopies * w + j) + (lane >> 4);
    const int c = (lane & 15) ^ (row & 15);
    // (only a batch below 32 rows has rows past M: its last row again)
    xoff[j] = (uint32_t)((MB == 1 ? min(row, M - 1) : row) * K * 2 + c * 16);
  }
  const int col = cols_in ? n0 + r : r;          // (columns past N compute, and store nothing)
  const uint32_t woff = (uint32_t)(col * 64 + h * 32);
  auto issue_x = [&](int g, int st, int j) {
    dma16_s(x + (size_t)(m0 + 16 * (j / 4)) * K + (size_t)g * kAwqGroup, xoff[j % 4],
            (bf16_t*)(lds + st * Sh::kX + (Sh::kCopies * w + j) * 1024));
  };
  struct Codes {
    u32x4 wd[2][2];
    uint32_t sc[2], z[2];
  };
  auto fetch = [&](int g, Codes& cd) {
    const char* qb = (const char*)(qw + (size_t)g * N * 16);
    const bf16_t* sb = scales + (size_t)g * N;
    const uint8_t* zb = zeros + (size_t)g * N;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
        cd.wd[nb][q] = *reinterpret_cast<const u32x4*>(qb + woff + nb * 2048 + q * 16);
      cd.sc[nb] = sb[col + 32 * nb];
      cd.z[nb] = zb[col + 32 * nb];
    }
  };

  f32x16 u[MB][2];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) u[a][b][j] = 0.f;
  float cref[2] = {1.f, 1.f};
  uint32_t nz[2] = {0, 0};                       // zero-point operands of the previous group

  char* const SP = lds + 2 * Sh::kX;

  Codes next;
#pragma unroll
  for (int j = 0; j < Sh::kCopies; ++j) issue_x(g_begin, 0, j);
  fetch(g_begin, next);
  for (int i = threadIdx.x; i < 2 * Sh::kSP / 16; i += (64 * NW))
    *reinterpret_cast<u32x4*>(SP + i * 16) = u32x4{0, 0, 0, 0};

  // u += (previous group's sums) (its -(128 + z) 2^e); pieces of slot `slot`
  auto zero_term = [&](int slot) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const bf16x8 v = as_bf16x8(*reinterpret_cast<const u32x4*>(
          SP + slot * Sh::kSP + (32 * mb + r) * 32 + h * 16));
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        const u32x4 b = {nz[nb], nz[nb], nz[nb], nz[nb]};
        u[mb][nb] = mfma32(v, as_bf16x8(b), u[mb][nb]);
      }
    }
  };

  for (int it = 0; it < n_groups; ++it) {
    // this group's copies have landed and every wave is done with the stage
    // that the next group's copies overwrite
    wait_vm<0>();
    __syncthreads();
    const Codes cd = next;
    const int g_next = g_begin + min(it + 1, n_groups - 1);   // (the last group again: unused)
    const char* SX = lds + (it & 1) * Sh::kX;
    auto a_op = [&](int row, int t) {
      return as_bf16x8(*reinterpret_cast<const u32x4*>(
          SX + row * 256 + (((2 * t + h) ^ (row & 15)) * 16)));
    };
    bf16x8 zp[MB], acur[MB], anxt[MB];
    const char* spr = SP + ((it + 1) & 1) * Sh::kSP + r * 32 + h * 16;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      zp[mb] = as_bf16x8(*reinterpret_cast<const u32x4*>(spr + mb * 1024));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acur[mb] = a_op(32 * mb + r, 0);
    // ---- the previous group's zero-point term (zero pieces before the first
    // group), beside the columns' constants and the first code operands ----
    float rho[2];
    uint32_t mask[2], magic[2];
    u32x4 bcur[2], bnxt[2];
    const u32x4 bz[2] = {{nz[0], nz[0], nz[0], nz[0]}, {nz[1], nz[1], nz[1], nz[1]}};
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      ColScale cs = col_scale_plain(cd.sc[nb], cd.z[nb]);
      rho[nb] = cref[nb] * __builtin_amdgcn_rcpf(cs.c);
      if (__builtin_expect(wave_any(!plain_scale(cd.sc[nb])), 0)) {
        asm volatile("");                        // (not executed and selected)
        cs = col_scale(cd.sc[nb], cd.z[nb]);
        rho[nb] = cs.mask == 0u ? 1.f : cref[nb] * __builtin_amdgcn_rcpf(cs.c);
        if (cs.mask == 0u) cs.c = cref[nb];
      }
      cref[nb] = cs.c;
      mask[nb] = in_vgpr(cs.mask);
      magic[nb] = in_vgpr(cs.magic);
      nz[nb] = cs.nz | (cs.nz << 16);
    }
    // pair p of the code operand of k-step t
    auto code_pair = [&](int nb, int t, int p) {
      return ((cd.wd[nb][t & 1][t >> 1] >> (4 * p)) & mask[nb]) | magic[nb];
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) {
      const int mb = i >> 1, nb = i & 1;
      u[mb][nb] = mfma32(zp[mb], as_bf16x8(bz[nb]), u[mb][nb]);
#pragma unroll
      for (int e = i * 16 / (2 * MB); e < (i + 1) * 16 / (2 * MB); ++e) {
        if (e < 8) bcur[e >> 2][e & 3] = code_pair(e >> 2, 0, e & 3);
        else bnxt[(e >> 2) & 1][e & 3] = code_pair((e >> 2) & 1, 1, e & 3);
      }
      if (nb == 1) anxt[mb] = a_op(32 * mb + r, 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- u <- u c / m, block by block under the MFMAs of k-steps 0 and 1 of
    // the block before ----
    auto rescale = [&](int i, int part) {
#pragma unroll
      for (int j = 8 * part; j < 8 * part + 8; ++j) u[i >> 1][i & 1][j] *= rho[i & 1];
    };
    float sums[Sh::kPer][2];
#pragma unroll
    for (int i = 0; i < Sh::kPer; ++i) sums[i][0] = sums[i][1] = 0.f;
    // sum unit i (even ones in steps 0-3, odd ones in 4-7): rows 32 (id / 2),
    // k-steps 4 (id % 2) + t % 4
    u32x4 sf[Sh::kPer];
    auto sum_read = [&](int t) {
#pragma unroll
      for (int i = 0; i < Sh::kPer; ++i)
        if ((i & 1) == (t >> 2)) {
          const int id = (w + NW * i) % Sh::kUnits;
          sf[i] = as_u32x4(a_op(32 * (id >> 1) + r, 4 * (id & 1) + (t & 3)));
        }
    };
    auto sum_add = [&](int t) {
#pragma unroll
      for (int i = 0; i < Sh::kPer; ++i)
        if ((i & 1) == (t >> 2)) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sums[i][e & 1] = dot2_ones(sf[i][e], sums[i][e & 1]);
        }
    };
    auto pieces = [&](int i) {
      const int id = w + NW * i;
      const float s = sums[i][0] + sums[i][1];
      const __bf16 p1 = (__bf16)s;
      const float d1 = s - (float)p1;
      const __bf16 p2 = (__bf16)d1;
      const __bf16 p3 = (__bf16)(d1 - (float)p2);
      const u32x2 pc = {(uint32_t)__builtin_bit_cast(uint16_t, p1) |
                            ((uint32_t)__builtin_bit_cast(uint16_t, p2) << 16),
                        (uint32_t)__builtin_bit_cast(uint16_t, p3)};
      // (an opaque lane: the address is formed here, not kept over the loop)
      const int ln = (int)in_vgpr(threadIdx.x) & 63;
      if (id < Sh::kUnits)
        *reinterpret_cast<u32x2*>(SP + (it & 1) * Sh::kSP + 1024 * (id >> 1) + 8 * (id & 1) +
                                  (ln & 31) * 32 + (ln >> 5) * 16) = pc;
    };
    rescale(0, 0);
    rescale(0, 1);
    bf16x8 a2[MB];
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) {
      const int mb = i >> 1, nb = i & 1;
      __builtin_amdgcn_sched_barrier(0);
      u[mb][nb] = mfma32(acur[mb], as_bf16x8(bcur[nb]), u[mb][nb]);
      if (i + 1 < 2 * MB) rescale(i + 1, 0);
      if (i == 0) sum_read(0);
      __builtin_amdgcn_sched_barrier(0);
      u[mb][nb] = mfma32(anxt[mb], as_bf16x8(bnxt[nb]), u[mb][nb]);
      if (i + 1 < 2 * MB) rescale(i + 1, 1);
      if (nb == 1) a2[mb] = a_op(32 * mb + r, 2);
      if (i == 2 * MB - 1) {
        sum_add(0);
        sum_read(1);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch(g_next, next);                         // (no earlier: registers)
    sum_add(1);
#pragma unroll
    for (int e = 0; e < 8; ++e) bcur[e >> 2][e & 3] = code_pair(e >> 2, 2, e & 3);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acur[mb] = a2[mb];
    // ---- k-steps 2 to 7: one MFMA, then a share of the next step's operands,
    // the sums and the next group's copies ----
#pragma unroll
    for (int t = 2; t < 8; ++t) {
      sum_read(t);
#pragma unroll
      for (int i = 0; i < 2 * MB; ++i) {
        const int mb = i >> 1, nb = i & 1;
        __builtin_amdgcn_sched_barrier(0);
        u[mb][nb] = mfma32(acur[mb], as_bf16x8(bcur[nb]), u[mb][nb]);
        if (t < 7) {
#pragma unroll
          for (int e = i * 8 / (2 * MB); e < (i + 1) * 8 / (2 * MB); ++e)
            bnxt[e >> 2][e & 3] = code_pair(e >> 2, t + 1, e & 3);
          if (nb == 1) anxt[mb] = a_op(32 * mb + r, t + 1);
        }
        if (i == 2 * MB - 1) sum_add(t);
        if (i < Sh::kCopies && t >= 2 && t < 6 && i * 4 / Sh::kCopies == t - 2)
          issue_x(g_next, (it + 1) & 1, i);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (Sh::kPer > 1 && t == 4) pieces(0);
      if (t < 7) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acur[mb] = anxt[mb];
        bcur[0] = bnxt[0];
        bcur[1] = bnxt[1];
      }
    }
#pragma unroll
    for (int i = 1; i < Sh::kPer; ++i) pieces(i);
    if constexpr (Sh::kPer == 1) pieces(0);
  }
  wait_vm<0>();                                  // (the last, unused copies)
  __syncthreads();
  zero_term((n_groups + 1) & 1);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int j = 0; j < 16; ++j) u[mb][nb][j] *= cref[nb];

  // ---- groups split over workgroups: fp32 partials (device-coherent stores,
  // another XCD may add them), then the last workgroup of the tile to arrive
  // reads all of them back (its own too), adds them in split order and leaves the
  // tile's counter at zero ----
  if constexpr (kSplit) {
    constexpr int kVals = MB * 32;               // values per lane
    const size_t per_split = (size_t)NW * 64 * kVals;
    float* mine = part + ((size_t)pid * splits + blockIdx.y) * per_split +
                  (size_t)w * 64 * kVals + 2 * lane;
    if (cols_in) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int j = 0; j < 16; j += 2)
            store_coherent2(mine + ((mb * 2 + nb) * 16 + j) * 64, u[mb][nb][j], u[mb][nb][j + 1]);
    }
    wait_all_memory();
    __syncthreads();
    int* flag = reinterpret_cast<int*>(lds);
    if (threadIdx.x == 0)
      *flag = __hip_atomic_fetch_add(arrivals + pid, 1, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int arrived = *flag;
    __syncthreads();                             // flag read: the LDS is free again
    if (arrived != splits - 1) return;
    if (threadIdx.x == 0)
      __hip_atomic_store(arrivals + pid, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // (the partials of four splits and one row block in flight at a time: a
    // load takes a round trip to the coherence point)
    const float* tile = part + (size_t)pid * splits * per_split + (size_t)w * 64 * kVals + 2 * lane;
    constexpr int kBatch = 4;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      float acc[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) acc[j] = 0.f;
      for (int s0 = 0; s0 < splits; s0 += kBatch) {
        float v[kBatch][32];
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
#pragma unroll
          for (int j = 0; j < 32; j += 2) {
            float p[2];
            load_coherent_vec<2>(tile + (size_t)min(s0 + b, splits - 1) * per_split +
                                     (mb * 32 + j) * 64, p);
            v[b][j] = p[0];
            v[b][j + 1] = p[1];
          }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
#pragma unroll
          for (int j = 0; j < 32; ++j) acc[j] += s0 + b < splits ? v[b][j] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < 32; ++j) u[mb][j >> 4][j & 15] = acc[j];
    }
  }

  // ---- output: transposed through LDS so that each lane stores 16 contiguous
  // bytes, 32 rows at a time ----
  if constexpr (!kSplit) __syncthreads();
  char* T = lds + w * 32 * kOutStride;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int row = 8 * (j >> 2) + 4 * h + (j & 3);
        *reinterpret_cast<__bf16*>(T + row * kOutStride + 2 * (32 * nb + r)) = (__bf16)u[mb][nb][j];
      }
    wave_lds_sync();
    if (cols_in) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int idx = 64 * i + lane;
        const int row = idx >> 3, ch = idx & 7;
        const int grow = m0 + 32 * mb + row;
        const u32x4 v = *reinterpret_cast<const u32x4*>(T + row * kOutStride + ch * 16);
        if (MB > 1 || grow < M) *reinterpret_cast<u32x4*>(y + (size_t)grow * N + n0 + 8 * ch) = v;
      }
    }
    wave_lds_sync();
  }
}

// ---------------------------------------------------------------------------
// Small batches (M <= 64), where streaming the codes from HBM is the cost.
// 16x16x32 MFMAs (16 rows per block: no padding rows for a decode batch of
// 16), one workgroup of W waves per 16 NB output columns (NB blocks of 16
// columns, which share each activation read) and split of the groups.  The
// waves form A column ranges of NB / A blocks (at most four: the conversion
// of the codes, about one VALU instruction per code, is what a wave's time
// goes to) by W / A group phases: wave w takes column range w % A and the
// groups [p R, p R + R) of the workgroup's G of phase p = w / A,
// R = ceil(G / (W / A)).
//
// X.  The waves of a phase first copy its groups' X (16-row blocks of 16 x 128,
// 4 KB each) into LDS with direct global -> LDS copies: each copy
// instruction moves four whole rows of a block (4 x 256 contiguous bytes, so
// no cache line is fetched twice), lane l of instruction i landing at
// position p = 64 i + l, which holds the 16-byte chunk j = (p % 16) ^ r of row
// r = p / 16.  The A operand of k-step t (lane (c, qq): row c, chunk 4 t + qq)
// is then one 16-byte LDS read at position 16 c + ((4 t + qq) ^ c): the 16
// lanes of a read group hit 16 different bank groups.  Rows past M read row
// M - 1 (their outputs are not stored).
//
// Codes.  Each wave streams its groups through a ring of register slots: the
// code words (16 contiguous bytes per lane and column block), scales and zero
// points of group i + depth, requested once group i is consumed (one row
// block) or as soon as it has taken its slot (more row blocks).
//
// Per group and 16-row block: P = sum_t X_t B_t over the 4 k-steps (B = the
// codes as bf16 128 + q), S = sum_t X_t 1 (a ones operand: lane (c, qq) gets
// the group sums of rows 4 qq .. 4 qq + 3, the rows of its outputs), and
// y += s (P - (128 + z) S) in fp32.  The sums of a column range's waves are
// added in LDS in phase (group) order.  With the groups split over
// workgroups, fp32 partials go out with
// device-coherent stores and the last workgroup of a column block to arrive
// (device-scope counter) adds them in split order and resets the counter.
// ---------------------------------------------------------------------------
namespace awq_sm {
constexpr int kXCap = 32;                        // 4 KB X blocks a workgroup can stage
constexpr int kLds = kXCap * 4096;
}  // namespace awq_sm

template <int MB, int NBW, int A, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void awq_gemm_sm_kernel(
    const bf16_t* __restrict__ x, const uint32_t* __restrict__ qw,
    const bf16_t* __restrict__ scales, const uint8_t* __restrict__ zeros,
    bf16_t* __restrict__ y, float* __restrict__ part, int* __restrict__ arrivals, int M, int N,
    int K, int splits) {
  using namespace awq_sm;
  static_assert(kWaves % A == 0, "the waves split into A column ranges");
  constexpr int NB = NBW * A;                      // 16-column blocks of the workgroup
  constexpr int kPhases = kWaves / A;              // waves per column range
  constexpr int kCols = 16 * NB;
  constexpr int kThreads = kWaves * 64;
  // Ring of register slots, 8 / (MB NBW) of them, at most four (more only
  // repeat the last group's loads).  One row block: at least
  // two, each refilled once its group is consumed; larger row blocks (whose
  // groups cost more to compute than to wait for): each refilled as soon as
  // it is taken (measured, 16 / 32 / 64 rows).
  constexpr bool kLate = MB == 1;
  constexpr int kDepth0 = 8 / (MB * NBW) > 4 ? 4 : (8 / (MB * NBW) > 1 ? 8 / (MB * NBW) : 1);
  constexpr int kDepth = kLate && kDepth0 < 2 ? 2 : kDepth0;
  constexpr int kOut = MB * NBW * 4;               // accumulator values per lane
  static_assert(kWaves * kOut * 64 * 4 <= kLds, "wave sums fit the X region");
  __shared__ __attribute__((aligned(16))) char lds[kLds];
  const int lane = threadIdx.x & 63, w = wave_id();
  const int ca = w % A, ph = w / A;                // column range, group phase
  const int c = lane & 15, qq = lane >> 4;
  const int n0 = kCols * blockIdx.x + 16 * NBW * ca + c;   // columns n0 + 16 nb
  const int groups = K / kAwqGroup;
  const int spl = blockIdx.y;
  const int per_wg = (groups + splits - 1) / splits;
  const int wg_g0 = spl * per_wg;
  const int wg_end = min(groups, wg_g0 + per_wg);
  const int per_wave = (per_wg + kPhases - 1) / kPhases;
  const int g0 = wg_g0 + ph * per_wave;
  const int ng = max(0, min(per_wave, wg_end - g0));
  const uint32_t kMask = in_vgpr(0x000F000Fu), kMagic = in_vgpr(0x43004300u);
  const int wpos = 8 * (qq & 1) + 4 * (qq >> 1);   // this lane's 4 words

  // ---- X of this phase's groups into LDS, the copies dealt over the phase's
  // A waves ----
  for (int ii = ca; ii < ng * MB * 4; ii += A) {
    const int blk = (g0 - wg_g0) * MB + (ii >> 2), part4 = ii & 3;   // (group, row block)
    const int gl = blk / MB, mb = blk % MB;
    const int p = 64 * part4 + lane;
    const int r = p >> 4, j = (p & 15) ^ r;
    const int row = min(16 * mb + r, M - 1);
    dma16(x + (size_t)row * K + (size_t)(wg_g0 + gl) * kAwqGroup + 8 * j,
          (bf16_t*)(lds + blk * 4096 + part4 * 1024));
  }

  struct Slot {
    u32x4 wd[NBW];
    uint32_t sbits[NBW], z[NBW];
  };
  // everything one group needs from HBM; raw values only (arithmetic on a
  // loaded value here would wait for the load)
  auto fetch = [&](int g, Slot& sl) {
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
      const size_t col = (size_t)g * N + n0 + 16 * nb;
      sl.wd[nb] = *reinterpret_cast<const u32x4*>(qw + col * 16 + wpos);
      sl.sbits[nb] = scales[col];
      sl.z[nb] = zeros[col];
    }
  };

  f32x4 yv[MB][NBW];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) yv[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  Slot ring[kDepth];
  const int g_last = g0 + max(ng, 1) - 1;
  if (ng > 0) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) fetch(min(g0 + d, g_last), ring[d]);
  }
  wait_vm<0>();                                    // this wave's X copies (and first codes) landed
  __atomic_signal_fence(__ATOMIC_SEQ_CST);         // no LDS read of X moves above the wait
  if constexpr (A > 1) __syncthreads();            // ... and those of the phase's other waves
  if (ng > 0) {
    const u32x4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    // Each pass takes kDepth groups, one per slot.  Refilled late (kLate),
    // there is no branch around a slot's loads, so the compiler's waits see
    // one order of requests and wait for a slot's own loads only, and the
    // refill lands in the slot's registers (no copies at the back edge,
    // which would wait for the loads just issued); passes past the wave's
    // last group recompute it and do not add it.  Refilled early, the loads
    // are unconditional too (clamped to the last group).
    for (int i0 = 0; i0 < ng; i0 += kDepth) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {
        const int i = i0 + d;
        if constexpr (!kLate) {
          if (i >= ng) break;
        }
        const int g = min(g0 + i, g_last);
        __builtin_amdgcn_sched_barrier(0);
        const Slot sl = ring[d];
        if constexpr (!kLate) {
          fetch(min(g + kDepth, g_last), ring[d]);
          __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 xa[4][MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const char* blk = lds + ((g - wg_g0) * MB + mb) * 4096;
#pragma unroll
          for (int t = 0; t < 4; ++t)
            xa[t][mb] = as_bf16x8(
                *reinterpret_cast<const u32x4*>(blk + 16 * (16 * c + ((4 * t + qq) ^ c))));
        }
        f32x4 p[MB][NBW], sx[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          sx[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int nb = 0; nb < NBW; ++nb) p[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          // one k-step at a time (converting every step's codes up front
          // would need their registers all at once)
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) sx[mb] = mfma16(xa[t][mb], as_bf16x8(ones), sx[mb]);
#pragma unroll
          for (int nb = 0; nb < NBW; ++nb) {
            const bf16x8 b = codes_to_bf16(sl.wd[nb][t], kMask, kMagic);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) p[mb][nb] = mfma16(xa[t][mb], b, p[mb][nb]);
          }
        }
        if (i < ng) {
#pragma unroll
          for (int nb = 0; nb < NBW; ++nb) {
            const float sc = bf16_to_f32(sl.sbits[nb]);
            const float nz = -(float)(128 + (int)sl.z[nb]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
              for (int j = 0; j < 4; ++j)
                yv[mb][nb][j] = fmaf(sc, fmaf(nz, sx[mb][j], p[mb][nb][j]), yv[mb][nb][j]);
          }
        }
        if constexpr (kLate) {
          __builtin_amdgcn_sched_barrier(0);
          fetch(min(g0 + i + kDepth, g_last), ring[d]);   // slot consumed: refill it
        }
      }
    }
  }


  // ---- the waves' sums, added in wave order (the X region is free) ----
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[(w * kOut + (mb * NBW + nb) * 4 + j) * 64 + lane] = yv[mb][nb][j];
  __syncthreads();
  constexpr int kTot = MB * NB * 4;                // output values per lane position
  constexpr int kPer = (kTot * 64 + kThreads - 1) / kThreads;   // outputs per thread
  float tot[kPer];
  int orow[kPer], ocol[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int idx = threadIdx.x + e * kThreads;     // (mb, nb, j, lane') of the tile
    const int l = idx & 63, j = (idx >> 6) & 3, nbg = (idx >> 8) % NB, mb = (idx >> 8) / NB;
    const bool have = idx < kTot * 64;
    orow[e] = have ? 16 * mb + 4 * (l >> 4) + j : M;
    ocol[e] = kCols * blockIdx.x + 16 * nbg + (l & 15);
    float acc = 0.f;
    if (have) {
      // the waves of column range nbg / NBW, in group order
      const int cw = nbg / NBW, nb = nbg % NBW;
#pragma unroll
      for (int v = 0; v < kPhases; ++v)
        acc += red[(((v * A + cw) * kOut) + (mb * NBW + nb) * 4 + j) * 64 + l];
    }
    tot[e] = acc;
  }
  if (splits == 1) {
#pragma unroll
    for (int e = 0; e < kPer; ++e)
      if (orow[e] < M) {
        const __bf16 o = (__bf16)tot[e];
        y[(size_t)orow[e] * N + ocol[e]] = __builtin_bit_cast(bf16_t, o);
      }
    return;
  }
  // ---- groups split over workgroups: fp32 partials (device-coherent stores,
  // another XCD may add them), then the last workgroup of the column block to
  // arrive adds them in split order and leaves its counter at zero ----
  __shared__ int flag;
#pragma unroll
  for (int e = 0; e < kPer; ++e)
    if (orow[e] < M) store_coherent(part + ((size_t)spl * M + orow[e]) * N + ocol[e], tot[e]);
  wait_all_memory();
  __syncthreads();
  if (threadIdx.x == 0)
    flag = __hip_atomic_fetch_add(arrivals + blockIdx.x, 1, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (flag != splits - 1) return;
  if (threadIdx.x == 0)
    __hip_atomic_store(arrivals + blockIdx.x, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // eight partials in flight at a time, added in split order
  float acc[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) acc[e] = 0.f;
  for (int s0 = 0; s0 < splits; s0 += 8) {
    float v[kPer][8];
#pragma unroll
    for (int e = 0; e < kPer; ++e)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int s2 = min(s0 + u, splits - 1);
        const int row = min(orow[e], M - 1);
        v[e][u] = load_coherent(part + ((size_t)s2 * M + row) * N + ocol[e]);
      }
#pragma unroll
    for (int e = 0; e < kPer; ++e)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < splits) acc[e] += v[e][u];
  }
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (orow[e] >= M) continue;
    const __bf16 o = (__bf16)acc[e];
    y[(size_t)orow[e] * N + ocol[e]] = __builtin_bit_cast(bf16_t, o);
  }
}

// RAG_AWQ_SM_NB / RAG_AWQ_SM_SPLITS (read at each call) fix the small-batch
// column blocks per workgroup (1, 2, 4 or 8) and the least split of the groups: a
// testing and tuning knob (any choice computes the same sums; only split
// counts change the fp32 addition order).
static int env_int(const char* name) {
  const char* e = std::getenv(name);
  return (e != nullptr && e[0] != 0) ? std::atoi(e) : 0;
}

// The tiles of awq_gemm_md_kernel and what they cost: `res` workgroups fit a CU
// (registers); one group step takes `step` us with one of them resident and
// step + (n - 1) more with n.
struct MdTile {
  int mb, nw, res;
  double step, more;
};
static constexpr MdTile kMdTiles[] = {{1, 4, 3, 0.84, 0.47}, {2, 4, 2, 1.13, 0.78},
                                      {3, 4, 2, 1.57, 1.15}, {4, 4, 2, 1.91, 1.56},
                                      {5, 4, 1, 2.66, 0},    {4, 8, 1, 3.35, 0}};

// Estimated time (us) of a launch: the busiest CU's n workgroups run in batches
// of `res`.  A split adds the partials' trip (written once, read once by the
// merging workgroups) and the merge's round trips.  Constants fitted to timings
// of every tile and split (M 33-4096, the 7B layers and generic shapes).
static double awq_md_cost(const MdTile& c, int64_t tiles, int splits, int groups_per_split,
                          int64_t mn) {
  const int64_t n = (tiles * splits + kAwqCus - 1) / kAwqCus;      // on the busiest CU
  const int64_t full = n / c.res, rest = n % c.res;
  const double step = full * (c.step + c.more * (c.res - 1)) +
                      (rest ? c.step + c.more * (rest - 1) : 0);
  double t = step * groups_per_split;
  if (splits > 1) t += 2.7 + 0.78e-6 * splits * mn + 0.52 * (splits - 1) * c.mb;
  return t;
}

// The best tile and split of awq_gemm_md_kernel in avail bytes of workspace:
// counters, then the partials of a split, in whole tiles (none unsplit).
static AwqPlan awq_plan_md(int M, int N, int K, size_t avail) {
  AwqPlan p{};
  p.groups = K / kAwqGroup;
  double best = 0;
  for (const MdTile& c : kMdTiles) {
    if (c.mb > 1 && 32 * c.mb > M) continue;
    const int tiles_m = (M + 32 * c.mb - 1) / (32 * c.mb);
    const int tiles_n = (N + 64 * c.nw - 1) / (64 * c.nw);
    const int64_t tiles = (int64_t)tiles_m * tiles_n;
    const size_t out = (size_t)tiles * (32 * c.mb) * (64 * c.nw) * sizeof(float);
    for (int want = 1; want <= 16 && want <= p.groups; ++want) {
      if (want > 1 && (tiles > awq_md::kMaxSplitTiles || c.nw != 4)) break;
      const int gps = (p.groups + want - 1) / want;
      const int splits = (p.groups + gps - 1) / gps;
      if (splits != want) continue;
      const size_t counters = splits > 1 ? kAwqCounterBytes : 0;
      const size_t part = splits > 1 ? splits * out : 0;
      if (counters + part > avail) continue;
      const double t = awq_md_cost(c, tiles, splits, gps, (int64_t)M * N);
      if (p.md_mb == 0 || t < best) {
        best = t;
        p.md_mb = c.mb;
        p.md_nw = c.nw;
        p.tiles_m = tiles_m;
        p.tiles_n = tiles_n;
        p.tiles = tiles;
        p.splits = splits;
        p.groups_per_split = gps;
        p.counter_bytes = counters;
        p.part_bytes = part;
      }
    }
  }
  p.tiles_per_xcd = (int)((p.tiles + kNumXcd - 1) / kNumXcd);
  return p;
}

static AwqPlan awq_plan_sm(int M, int N, int K) {
  AwqPlan p{};
  p.groups = K / kAwqGroup;
  const size_t up = 255;
  // Small batches: a workgroup stages X of at most kXCap 16-row blocks, so
  // the groups are split at least groups * MB / kXCap ways, and no further:
  // the merge of a split (coherent partial stores, arrival count, reloads)
  // costs more than the CUs a smaller grid leaves idle (the 7B o_proj at 16
  // rows: 6.5 us on 128 workgroups, 7.4 us split in two on 256).  The column
  // blocks per workgroup are the fewest (1, 2, 4, 8) for which the workgroups
  // fit one per CU (the 7B o_proj at 16 rows: 1 block, 256 workgroups, 5.0 us
  // against 6.0 us for 2 blocks on 128), else 8 (each workgroup copies X for
  // its groups: wider column tiles read it fewer times; the 7B gate_up_proj
  // at 64 rows, 47 us against 76 us with 2 blocks).
  p.tiles_m = 1;
  p.sm_mb = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
  const int min_splits = (p.groups * p.sm_mb + awq_sm::kXCap - 1) / awq_sm::kXCap;
  p.sm_nb = 8;
  for (int nb : {1, 2, 4, 8}) {
    if (N % (16 * nb) != 0) continue;
    if ((int64_t)(N / (16 * nb)) * min_splits <= kAwqCus) {
      p.sm_nb = nb;
      break;
    }
  }
  if (const int nb = env_int("RAG_AWQ_SM_NB"); (nb == 1 || nb == 2 || nb == 4 || nb == 8) && N % (16 * nb) == 0)
    p.sm_nb = nb;
  p.tiles_n = N / (16 * p.sm_nb);
  // A waves share the column blocks, at most four blocks each and
  // MB * NB / A <= 8 (registers): eight blocks at 16 rows (the 7B
  // gate_up_proj) go to two waves of four, each taking a quarter of the
  // groups (14.1 us against 15.3 us for eight waves over all eight blocks;
  // two blocks per wave, 14.8 us; one, 16.2 us)
  p.sm_a = p.sm_nb / std::min({p.sm_nb, 4, 8 / p.sm_mb});
  int splits = min_splits;
  if (const int sp = env_int("RAG_AWQ_SM_SPLITS"); sp > 0) splits = std::max(min_splits, sp);
  splits = std::max(1, std::min(splits, p.groups));
  p.groups_per_split = (p.groups + splits - 1) / splits;
  p.splits = (p.groups + p.groups_per_split - 1) / p.groups_per_split;
  p.tiles = (int64_t)p.tiles_n * p.splits;
  if (p.splits > 1) {
    // arrival counters first: zero-filled once by the caller, left zero by
    // every call
    p.counter_bytes = kAwqCounterBytes;
    p.part_bytes = ((size_t)p.splits * M * N * sizeof(float) + up) & ~up;
  }
  return p;
}

AwqPlan awq_plan(int M, int N, int K, size_t avail) {
  if (M > 64) return awq_plan_md(M, N, K, avail);
  // awq_gemm_sm_kernel for up to 64 rows except where its tiles are the slower
  // ones: 33-64 rows of a layer above the 7B o_proj's size (7B gate_up at 64
  // rows 49 us against 29, o_proj 14.0 against 15.1), 17-32 rows of a wide one
  // (gate_up at 32 rows 27 against 20, N = 12288 15.7 either way).
  const bool knobs = env_int("RAG_AWQ_SM_NB") > 0 || env_int("RAG_AWQ_SM_SPLITS") > 0;
  // Where the small kernel needs no split and a workgroup a CU it stays the faster
  // one, whatever the width (17 rows: N = 32768, K = 1024 8.1 us against 10.8, 28672
  // x 2048 11.0 against 15.4; the shortest K the other way, 28672 x 128 4.3 against
  // 3.7).  Over 480 shapes of 17-64 rows the choice is at most 4% slower than the
  // small kernel, which is up to twice as slow as the choice.
  const AwqPlan sm = awq_plan_sm(M, N, K);
  const bool one_wave =
      sm.splits == 1 && sm.tiles_n <= kAwqCus && K >= (M > 32 ? 1024 : 512);
  const bool wide = !one_wave && ((M > 32 && (int64_t)N * K >= (int64_t)4608 * 4096) ||
                                  (M > 16 && N > 16384));
  // (more column blocks than counters: the row-tiled kernel has tiles enough
  // without a split)
  if (sm.splits > 1 && sm.tiles_n > kAwqCounters) return awq_plan_md(M, N, K, avail);
  auto fits = [avail](const AwqPlan& p) { return p.counter_bytes + p.part_bytes <= avail; };
  if (wide && !knobs) {
    const AwqPlan md = awq_plan_md(M, N, K, SIZE_MAX);
    if (fits(md)) return md;
  }
  // Up to 16 rows the small kernel's split needs its workspace, as it always has
  // (a call that brings less is refused); more rows fall back to the row-tiled
  // kernel in what there is.
  if (fits(sm) || M <= 16 || knobs) return sm;
  return awq_plan_md(M, N, K, avail);
}

hipError_t launch_awq_gemm(const AwqArgs& a, const AwqPlan& p, hipStream_t stream) {
  char* ws = static_cast<char*>(a.workspace);
  const bf16_t* x = (const bf16_t*)a.x;
  const uint32_t* qw = (const uint32_t*)a.qweight;
  const bf16_t* sc = (const bf16_t*)a.scales;
  bf16_t* y = (bf16_t*)a.y;
  int* counters = reinterpret_cast<int*>(ws);
  float* part = reinterpret_cast<float*>(ws + p.counter_bytes);
  if (p.md_mb > 0) {
    const dim3 grid((unsigned)(p.tiles_per_xcd * kNumXcd), (unsigned)p.splits);
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(p.md_nw * 64), 0, stream, x, qw, sc, a.zeros, y,
                         part, counters, a.M, a.N, a.K, p.groups_per_split, p.splits, p.tiles_m,
                         p.tiles_n, p.tiles_per_xcd);
    };
    const bool split = p.splits > 1;
    switch (p.md_mb * 10 + p.md_nw) {
      case 14: split ? go(awq_gemm_md_kernel<1, 4, true>) : go(awq_gemm_md_kernel<1, 4, false>); break;
      case 24: split ? go(awq_gemm_md_kernel<2, 4, true>) : go(awq_gemm_md_kernel<2, 4, false>); break;
      case 34: split ? go(awq_gemm_md_kernel<3, 4, true>) : go(awq_gemm_md_kernel<3, 4, false>); break;
      case 44: split ? go(awq_gemm_md_kernel<4, 4, true>) : go(awq_gemm_md_kernel<4, 4, false>); break;
      case 54: split ? go(awq_gemm_md_kernel<5, 4, true>) : go(awq_gemm_md_kernel<5, 4, false>); break;
      case 48: go(awq_gemm_md_kernel<4, 8, false>); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  if ((int64_t)p.groups_per_split * p.sm_mb > awq_sm::kXCap) return hipErrorInvalidValue;
  const dim3 grid((unsigned)p.tiles_n, (unsigned)p.splits), block(512);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, x, qw, sc, a.zeros, y, part, counters,
                       a.M, a.N, a.K, p.splits);
  };
  switch (p.sm_mb * 100 + p.sm_nb * 10 + p.sm_a) {
    case 121: go(awq_gemm_sm_kernel<1, 2, 1, 8>); break;
    case 111: go(awq_gemm_sm_kernel<1, 1, 1, 8>); break;
    case 211: go(awq_gemm_sm_kernel<2, 1, 1, 8>); break;
    case 411: go(awq_gemm_sm_kernel<4, 1, 1, 8>); break;
    case 141: go(awq_gemm_sm_kernel<1, 4, 1, 8>); break;
    case 182: go(awq_gemm_sm_kernel<1, 4, 2, 8>); break;
    case 221: go(awq_gemm_sm_kernel<2, 2, 1, 8>); break;
    case 241: go(awq_gemm_sm_kernel<2, 4, 1, 8>); break;
    case 282: go(awq_gemm_sm_kernel<2, 4, 2, 8>); break;
    case 421: go(awq_gemm_sm_kernel<4, 2, 1, 8>); break;
    case 442: go(awq_gemm_sm_kernel<4, 2, 2, 8>); break;
    case 484: go(awq_gemm_sm_kernel<4, 2, 4, 8>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rag
