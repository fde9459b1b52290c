// Host-side launch descriptors of the group-quantized int4-weight GEMM
// (internal; the public ABI is include/rag_attn.h).
#pragma once

#include <hip/hip_runtime.h>

#include <stddef.h>
#include <stdint.h>

namespace rag {

// Arrival counters at a workspace's start, one per column block or output tile
// of a split launch, at most: the same bytes for every call, as the partials
// behind them keep what the last call wrote and calls of any layer and batch
// may follow each other in one workspace.
constexpr int kAwqCounters = 16384;
constexpr size_t kAwqCounterBytes = kAwqCounters * sizeof(int);

struct AwqArgs {
  const void* x;                // bf16 [M, K]
  const int32_t* qweight;       // packed codes [K/128][N][16]
  const void* scales;           // bf16 [K/128, N]
  const uint8_t* zeros;         // [K/128, N]
  void* y;                      // bf16 [M, N]
  void* workspace;
  int M, N, K;
};

struct AwqPlan {
  int md_mb;                    // awq_gemm_md_kernel: 32-row blocks per tile (0: the small one)
  int md_nw;                    // its waves, 64 columns each
  int groups, splits, groups_per_split;
  int tiles_m, tiles_n, tiles_per_xcd;
  int sm_mb;                    // small batches: 16-row blocks (1, 2 or 4)
  int sm_nb;                    // small batches: 16-column blocks per workgroup
  int sm_a;                     // small batches: waves across the columns (NB / A blocks each)
  int64_t tiles;
  size_t counter_bytes;         // arrival counters (at the workspace's start), then
  size_t part_bytes;            // the partials of a split over the groups
};

// The launch of a call that has avail bytes of workspace; with more than 16 rows
// it fits whatever they are.
AwqPlan awq_plan(int M, int N, int K, size_t avail = SIZE_MAX);
hipError_t launch_awq_gemm(const AwqArgs& a, const AwqPlan& plan, hipStream_t stream);

}  // namespace rag
