// Internal interface between the C ABI (capi.cpp) and the HIP launchers
// (kernels.hip).  Not installed; not part of the public ABI.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace fqi {

constexpr int kTileK = 128;     // K side of a dense/sparse tile = quantisation group
constexpr int kTileN = 64;      // N side of a Tile-COO tile = widest output strip
constexpr int kMaxM = 128;      // rows the kernels support
constexpr int kSlabM = 32;      // rows one workgroup computes (two 16-row MFMA blocks)
constexpr int kMaxBuckets = 256;
constexpr int kXStride = 136;   // LDS row stride (elements) of a staged 128-wide X slice
constexpr int kGatherMaxM = 1;  // up to this M the sparse path gathers X in LDS; above, MFMA
constexpr int kGatherLimitM = 4; // rows the gather mapping can stage at all
constexpr int kImageBytes = 16384;   // one wave's B-operand image of a 128 x 64 tile
// The workspace starts with a fixed counter region (one uint32 per output
// strip, zero between calls) so that a workspace shared by problems of
// different shapes never finds partial sums where a counter is expected.
constexpr size_t kCounterRegion = 256 * 1024;
constexpr int kMaxStrips = int(kCounterRegion / 4);
// Static device scratch of the allocation-free entry point: the counter
// region followed by 8 MiB of split-K partial sums.  On the Llama-3-8B and -70B
// linears the strip kernel needs up to 4 MiB of them, the row-block kernel all
// 8 (14336 x 4096 above 32 rows): where it splits, its 256 workgroups of 32 KiB
// each are that much, and a launch that would need more is not made
// (kRowsPartialLimit).
constexpr size_t kScratchBytes = kCounterRegion + (size_t(8) << 20);

// The row-block kernel (rows.hip) serves more rows than this, with at least so
// many tiles per workgroup and partial sums that the static scratch holds.
constexpr int kRowsMinM = 16;
constexpr int kRowsMinTiles = 14;
constexpr double kRowsMinFill = 0.65; // of the rounds of workgroups, with more than one
constexpr int kRowsMaxGroups = 160;   // of the largest tile, with 64-row blocks
constexpr int kRowsMaxGroups32 = 64;  // the same with 32-row blocks: one load's worth
constexpr size_t kRowsPartialLimit = kScratchBytes - kCounterRegion;

// Launch plan of one matmul kernel.  The Tile-COO decides between the kernels,
// but no launch needs more workspace than fq_workspace_bytes finds from
// (M, K, N, split_k) alone, so the workspace can be sized before the Tile-COO
// exists.
struct Plan {
  int M, K, N;
  int MB;            // 16-row MFMA blocks per slab: 1 (M <= 16) or 2
  int n_slabs;       // 32-row slabs of M, one workgroup set each
  int slab_M;        // rows per slab: min(M, 32)
  int MODE;          // sparse mapping: 0 LDS gathers (M <= kGatherMaxM), 1 MFMA
  int NCB;           // 16-column MFMA blocks per strip: 2 (32-column strips) or 4 (64)
  int n_strips;      // N / (16 NCB)
  int T;             // tiles per strip, K / 128
  int S;             // K ranges per strip (explicit split-K); 1 under Stream-K
  int NW;            // dense (or dense and outlier) waves per workgroup: 4 or 8
  int NWS;           // outlier waves beside them (warp specialisation), 0 or NW / 2
  int stream;        // 1: Stream-K schedule, 0: uniform split-K
  int G;             // workgroups per slab
  int C;             // partial-sum slots per strip (most contributors to one strip)
  int B;             // buckets per tile
  int XS;            // row-wise X loads per tile through the LDS stage: 0, or 1, 2, 4 (ceil(M/4))
  int BK;            // 1: a dense wave loads the scales and zero-points of all its tiles at once
  int64_t max_tile_groups;   // the caller's largest group count of a tile
  int DV;            // 1: dense products by VALU dot products instead of MFMA (one row; ablation)
  // dynamic LDS layout, bytes: one slot per wave (X slice or B-operand
  // image), then the gather-mode sparse output buffers or the X stages
  size_t slot_bytes, off_shc, off_flag, off_trash, off_xs, lds_bytes;
  // workspace layout, bytes: counters at 0, partial sums at kCounterRegion
  // (ws_bytes: of whichever kernel runs; strip_ws_bytes: of the strip kernel)
  size_t partial_bytes, ws_bytes, strip_ws_bytes;
  // the row-block kernel's launch (rows.hip), where it is the one to run:
  // 32-row blocks per workgroup (0: the strip kernel runs), row blocks of M,
  // K ranges and workgroups per row block
  int rows_RB, rows_blocks, rows_S, rows_G;
  size_t rows_partial_bytes;
};

// Schedule options of make_plan (bit set).
constexpr int kOptStreamK = 1;     // Stream-K ranges instead of uniform split-K (split_k == 0)
constexpr int kOptFourWaves = 2;   // never eight waves per workgroup
constexpr int kOptStrip32 = 4;     // 32-column strips (MFMA outlier mapping, no Stream-K)
constexpr int kOptStrip64 = 8;     // 64-column strips
constexpr int kOptSparseWaves = 16;   // warp specialisation: outlier waves beside the dense waves
constexpr int kOptDenseValu = 32;     // dense products by VALU dot products (M == 1, MFMA mapping)

// Returns false when (M, K, N) is outside what the kernels implement.
// mode: -1 picks the sparse mapping by M, 0 forces gathers, 1 forces MFMA.
// n_groups: the Tile-COO's groups (a fused call with none runs dense only).
bool make_plan(int M, int K, int N, int split_k, bool dense, bool sparse, int B, int64_t n_groups,
               int64_t max_tile_groups, Plan* plan, int mode = -1, int opts = 0);

struct MatmulPtrs {
  const uint16_t* X;
  const uint32_t* Wq;
  const uint16_t* scales;
  const uint32_t* zeros;
  const uint32_t* tile_indptr;
  const uint16_t* bucket_info;
  const uint32_t* packed;
  int64_t n_groups;
  const float* y_addend;   // fp32 [M][N] added before the output is written, or null
  void* Y;
  int y_f32;
  void* workspace;
};

// Loads of 64 outlier groups a tile issues (kernels.hip): 1, or 2 where the
// tiles are full; 0 without outliers.  Only the MFMA mapping under uniform
// split-K without outlier waves, and the row-block kernel, have the second.
int group_loads(const Plan& plan, int64_t n_groups, bool sparse);

// Adds the row-block kernel's launch to a plan made without a forced split or
// schedule switch, where that kernel is the faster one (rows.hip).
void plan_rows(Plan* plan, bool outliers);
int launch_rows(const Plan& plan, const MatmulPtrs& p, bool sparse, bool two_group_loads,
                void* stream);
size_t rows_lds_bytes(const Plan& plan);

#ifdef FQ_WAVE_STAMPS
// Instrumented build: the current device's stamps, kMaxStampWaves x 4 (null: none).
constexpr int kMaxStampWaves = 8192;
uint64_t* wave_stamps_address();
#endif

// Enqueues one matmul kernel; returns a hipError_t value (0 on success).
int launch_matmul(const Plan& plan, const MatmulPtrs& p, bool dense, bool sparse, void* stream);

// The calling thread's current device's copy of the static scratch array
// (kScratchBytes, 256-byte aligned).  Set up once per device: the array's
// device address is looked up and its counter region cleared by a kernel on
// `stream`.  Returns a hipError_t value (0 on success).
int scratch_for_current_device(void** ptr, void* stream);

// Enqueues the group decoder over every group; returns a hipError_t value.
int launch_decode(const uint32_t* tile_indptr, int64_t n_tiles, const uint32_t* packed,
                  int64_t n_groups, int kt_count, int k_tile, int n_tile, int32_t* k_out,
                  int32_t* n_out, uint16_t* v_out, void* stream);

}  // namespace fqi
