// Projection kernel interface (see k_gemm.hip).
#pragma once

#include "internal.hpp"

namespace vsk {

enum { EPI_RESID = 0, EPI_QKV = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };

struct GemmArgs {
  const uint32_t __attribute__((ext_vector_type(4)))* W;  // packed tiles
  const uint32_t __attribute__((ext_vector_type(4)))* X;  // activation frags
  int Kt;       // K / 32
  int N;        // output columns
  int R;        // valid rows
  int Rg;       // 16-row groups of the X frag buffer
  float* x;          // RESID: fp32 residual [R][N], x += y
  double* ssq_out;   // RESID: partial sums of x^2 of the updated rows [R][n_groups]
  uint16_t* out;  // QKV: q [R][Nq]; SWIGLU: frags (out_Rg); LOGITS: logits [R][N]
  int out_Rg;
  uint16_t* pool;  // QKV: KV pool
  int layer, n_blocks, Hkv, hd, Nq, Nkv;
  const int32_t* slot;
  const int32_t* pos;
  const float2* rope;  // [max_pos][hd/2] (cos, sin)
  float* am_val;       // LOGITS: [n_groups][R]
  int* am_idx;
  float* ypart;  // RESID with K split over workgroups: y[split][R][N] instead of x += y
  const int* count;  // nullable: rows of this launch read on the device (<= R; a cohort's size)
  int xcd_remap;     // row-tiled passes: row tiles of one N group on one XCD at the same time
};

struct GemmPlan {
  int mg = 1;        // 16-row groups per tile
  int m_tiles = 1;   // tiles along the rows
  int n_groups = 1;  // workgroups along N (also the number of x^2 partials a RESID emits)
  int nt = 1;        // N tiles per wave
  int wn = 1;        // waves side by side along N
  int ksplit = 1;    // RESID: workgroups along K, their products added by k_resid_norm
  bool tiled = false;  // k_gemm_tiled (17..64 rows): n_groups of nt x wn column tiles
  bool xl = false;   // X chunks staged in LDS by a loader wave, shared by the compute waves
};

constexpr int kMaxResidSplits = 8;
constexpr int kResidTargetWgs = 0;  // default split-K target of the residual projections (0: no split)
constexpr int kTiledGroups = 4;       // 16-row groups of a k_gemm_tiled launch
constexpr int kTiledTargetWgs = 256;  // default split-K target at 17..64 rows: one round of compute units
constexpr int kQkvTargetWgs = 192;  // and of QKV in the layouts of k_gemm
constexpr int kRowTiledSplitBelow = 128;  // row-tiled residual projections split K at or below these workgroups
constexpr int kRowTiledTarget = 256;      // into as many splits as stay within this many workgroups
constexpr int kComputeUnits = 256;        // MI355X: 8 XCDs x 32 compute units

// shape: launch shape for 4 or 8 row groups (0 default; see k_gemm.hip)
// resid_target: workgroups a residual projection's K split aims for (-1: no
// split; 0: the layout's default -- kTiledTargetWgs in k_gemm_tiled, 384 (192
// at 4 row groups) with X in LDS, 192 for the two-tile layout of the down
// projection at <= 16 rows, else kResidTargetWgs)
// row_tile: 16-row groups per tile of a row-tiled projection other than the
// lm_head (0: chosen from the launch rounds; 6, 7, 8 or 11: that height)
GemmPlan plan_gemm(int N, int K, int R, int epi, int shape = 0, int resid_target = 0, int row_tile = 0);
// The plan of a projection of 17..64 rows in k_gemm_tiled.  target: for EPI_RESID
// the workgroups a K split may reach (0: no split).  Of 64, 128 and 256 columns
// per workgroup it takes the one whose compute units move the fewest bytes
// (rounds x K steps x (row groups + column tiles)), which ranks the layouts as
// measured: 28672 x 4096 at 64 rows 64 / 128 / 256 columns 46.5 / 39.5 / 58.0
// us, 16384 x 3072 18.9 / 25.5 / 40.1, 32000 x 4096 at 37 rows 46.4 / 42.7 /
// 59.6, 128256 x 3072 at 64 rows 159 / 148 / 139.
GemmPlan plan_tiled(int N, int K, int R, int epi, int target);
hipError_t launch_gemm_tiled(const GemmArgs& a, const GemmPlan& p, int epi, hipStream_t s, const LaunchEvents& ev);
hipError_t launch_gemm(GemmArgs a, const GemmPlan& p, int epi, hipStream_t s, LaunchEvents ev = {});
// QKV with K split: add the `splits` products in a.ypart and apply the QKV
// epilogue (a as for the QKV projection, with N = Nq + 2 Nkv).
hipError_t launch_qkv_reduce(const GemmArgs& a, int splits, hipStream_t s);

}  // namespace vsk
