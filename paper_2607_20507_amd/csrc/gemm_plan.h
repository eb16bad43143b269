// Host-side choice of a bf16 projection's kernel, tile shape and K split.
#pragma once

#include <cstddef>

#include "gemm.h"

namespace spec {

// gemm_mfma2_bf16: 32 mtw rows x 32 ntw W rows per workgroup.
struct Mfma2Shape {
  int mtw, ntw;
};

// gemm_mfma3_bf16: tiles of 16 kM3MB rows x 64 kM3NB W rows, operands kM3D
// k-steps ahead.
constexpr int kM3MB = 12, kM3NB = 4, kM3D = 4;
// Small form: 64-row tiles (MB 4) of 64 NB W rows, K split to fill the CUs,
// for the drafter's and the target's 41-128-row projections, where every
// workgroup streams all of X: a 64-row tile streams 4 KB of X per k-step
// through LDS against the 16 KB of the 192-row form.
constexpr int kM3sMB = 4;

struct Mfma3Plan {
  int MT, NT, S, k_len;
  int nb;  // 0: the 192 x 256 form; else the small form with NB = nb
};

// gemm_mfma4_bf16: operands of W and X in flight, in k-steps; row tiles per
// group.
constexpr int kM4DW = 4, kM4DX = 8, kM4Group = 4;

struct M4Tiles {
  int MT, NT, S, k_len;  // row tiles, W tiles, K splits and their length
};

// Estimated time in us of one kernel form.  A workgroup's k-step takes `step`
// plus the 2-norm of three streams: its MFMAs (`mfma` us per 1000 MFMA
// cycles), the rows of X and W that it takes in (`in` us per 1000) and the
// launch's W tiles (`w` us per MB); a launch `start`, a round of workgroups
// `round`.
struct FormCost {
  double mfma, step, in, w, start, round;
};
struct M4Shape {
  int mb, nb, occ;  // tile 16 mb rows x 64 nb W rows, workgroups per CU
  FormCost cost;
};
// 256 x 256 down to 64 x 128: fewer bytes per flop against more workgroups.
constexpr M4Shape kM4Shapes[] = {{16, 4, 1, {0.531, 0.025, 0.0, 0.0675, 3.56, 8.82}},
                                 {16, 3, 1, {0.609, 0.024, 0.0, 0.0557, 4.84, 4.65}},
                                 {12, 4, 1, {0.524, 0.111, 0.0, 0.0577, 6.77, 2.70}},
                                 {8, 4, 1, {0.769, 0.0, 0.0, 0.0602, 5.92, 1.81}},
                                 {8, 2, 2, {0.723, 0.058, 0.0, 0.0674, 5.26, 1.07}},
                                 {4, 2, 2, {0.769, 0.091, 0.0, 0.0841, 5.49, 0.0}}};
constexpr int kM4Shapes_n = sizeof(kM4Shapes) / sizeof(kM4Shapes[0]);

// What follows the GEMM: nothing, the RMSNorm (which a split's second pass
// applies), or rope_kv (which sums a split's partials).
enum class Tail { kNone, kNorm, kRope };

struct MfmaPlan {
  enum { kM2, kM3, kM4 } kernel = kM2;
  Mfma2Shape m2{2, 2};
  Mfma3Plan m3{};
  int shape = -1;  // gemm_mfma4_bf16: index into kM4Shapes
  M4Tiles tl{};
};

// The kernel of a projection that use_mfma sends to the MFMA kernels; m4: the
// outputs and partials are aligned for gemm_mfma4_bf16.
MfmaPlan plan_mfma(int R, int N, int K, int epi, size_t ws_bytes, bool m4, Tail tail);

int mfma2_splits(int MT, int NT, int R, int Nw, int K, size_t ws_bytes, int* k_len);

bool use_mfma(int R, int Nw, int K);

}  // namespace spec
