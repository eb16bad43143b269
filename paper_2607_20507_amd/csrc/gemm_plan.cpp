// Which kernel, tile shape and K split a bf16 projection takes.

#include <algorithm>
#include <cmath>

#include "gemm_plan.h"

namespace spec {

// Skinny (weight streaming, X re-read per 16-feature tile) or MFMA tiles (X
// staged once per workgroup tile): measured at 9..64 rows on the 8B- and
// 1B-shaped projections, the MFMA kernel wins above 40 rows, above 12 rows
// for long reductions (K >= 8192) and the 128256-row LM heads, and above 24
// rows for projections of >= 16M weights.
bool use_mfma(int R, int Nw, int K) {
  if (R > 40) return true;
  if (R > 12 && (K >= 8192 || Nw >= 65536)) return true;
  return R > 24 && static_cast<double>(Nw) * K >= 16.0 * (1 << 20);
}

// Split-K of gemm_mfma2_bf16: grids under 192 tiles are split so that
// tiles x splits fills the 256 CUs about once (k-splits multiples of 128,
// partials within the workspace).  Returns S and the k-split length.
int mfma2_splits(int MT, int NT, int R, int Nw, int K, size_t ws_bytes, int* k_len) {
  int S = 1;
  if (ws_bytes && MT * NT < 192) {
    S = std::max(1, std::min(8, 256 / (MT * NT)));
    while (S > 1 && static_cast<size_t>(S) * R * Nw * sizeof(float) > ws_bytes) --S;
  }
  *k_len = ((K + S - 1) / S + 127) / 128 * 128;
  return (K + *k_len - 1) / *k_len;
}

namespace {

// Tile shape of gemm_mfma2_bf16: rows per workgroup 32 MTW (64 .. 256) and W
// rows per workgroup 32 NTW (64 .. 256), the pair with the least estimated
// time in a cost model fitted (least squares, median error 10%) to measured
// launches of every shape at 64, 128 and 364 rows of the 8B/1B-shaped
// projections: per-step terms for the MFMAs and the LDS loads of a
// workgroup, times the k-steps and the rounds of workgroups over the 256
// CUs, plus the split-K partial traffic.  Wide tiles waste rows or feed too
// few CUs on small problems; narrow ones reload X and W more often.  A split
// SwiGLU pays its second pass as a launch of its own (≈ 6 us; the residual-add
// and QKV reductions ride on launches that follow anyway: the RMSNorm and the
// rotary embedding): with it the 41-128-row gate/up projections take narrow
// unsplit tiles (41-row 1B-shaped gate/up 19.6 -> 16.9 us, 8B-shaped
// 40.8 -> 36.2 us).
Mfma2Shape mfma2_shape(int R, int N, int Nw, int K, size_t ws_bytes, bool swiglu) {
  Mfma2Shape best{2, 2};
  double best_t = 1e300;
  for (int mtw : {2, 4, 6, 8}) {
    if (32 * mtw > 2 * R + 64) continue;  // tiles far taller than R
    for (int ntw : {2, 4, 8}) {
      const int MT = (R + 32 * mtw - 1) / (32 * mtw), NT = (Nw + 32 * ntw - 1) / (32 * ntw);
      int k_len = K;
      const int S = mfma2_splits(MT, NT, R, Nw, K, ws_bytes, &k_len);
      const double rounds = (MT * NT * S + 255) / 256;  // whole rounds of workgroups over the CUs
      const double steps = rounds * (k_len / 32);
      const double red_mb = S > 1 ? (S + 1.0) * R * N * 4.0 / 1e6 : 0.0;
      const double t = 0.0119 * steps * mtw * ntw + 0.0056 * steps * (32.0 * (mtw + ntw)) * 64.0 / 1024.0 +
                       0.0574 * steps + 0.3048 * red_mb + (S > 1 ? (swiglu ? 6.0 : -6.41) : 0.0);
      if (t < best_t) {
        best_t = t;
        best = {mtw, ntw};
      }
    }
  }
  return best;
}

// gemm_mfma3_bf16's shapes against gemm_mfma2_bf16: the 192-row form for
// residual adds with K >= 8192 whose grid splits K (the 364-row down projection
// 76 -> 64 us), and for SwiGLU from 160 rows and store-only projections of
// 65536+ rows in one pass when the tiles fill the 256 CUs at least 3 / 4 of the
// way (364-row gate/up 114 -> 97 us); the 64-row form below 129 rows and for
// some residual adds.  Above 128 rows plan_mfma weighs the result against
// gemm_mfma4_bf16.

// NB of the small form for a projection of R rows, or 0 where
// gemm_mfma2_bf16 is used (more than 128 rows; the 65536+-row LM heads).  From
// a sweep of NB in {1, 2, 4} against gemm_mfma2_bf16 over 13-150 rows of the
// 8B- and 1B-shaped projections: a residual add or plain store wants about 64
// tiles (K split 4 ways), so the narrowest W tile with at most 64 tiles; a
// SwiGLU, whose split costs a launch of its own, the widest tile that still
// fills 192 CUs unsplit, else NB = 2.  Measured against gemm_mfma2_bf16:
// 8B-shaped O projection at 41 rows 13.6 -> 11.3 us, gate/up at 96 rows 47.0 ->
// 37.9 us, down at 96 rows 31.4 -> 27.6 us; 1B-shaped down at 41 rows 13.5 ->
// 12.3 us, gate/up at 78 rows 20.1 -> 17.6 us; elsewhere within a few percent.
int mfma3_small_nb(int R, int Nw, int K, int epi) {
  (void)K;
  if (R > 128 || Nw >= 65536) return 0;
  const int MT = (R + 16 * kM3sMB - 1) / (16 * kM3sMB);
  auto tiles = [&](int nb) { return MT * ((Nw + 64 * nb - 1) / (64 * nb)); };
  if (epi == kEpiSwiGLU) return tiles(4) >= 192 ? 4 : 2;
  for (int nb : {1, 2}) if (tiles(nb) <= 64) return nb;
  return 4;
}

bool use_mfma3(int R, int Nw, int K, int epi, size_t ws_bytes, Mfma3Plan* plan) {
  if (K % (32 * kM3D)) return false;
  if (static_cast<double>(Nw) * K >= 2147483648.0 || static_cast<double>(R) * K >= 2147483648.0) return false;
  if (R < 160) {
    const int nb = ws_bytes ? mfma3_small_nb(R, Nw, K, epi) : 0;
    if (nb == 0 || (epi == kEpiSwiGLU && nb % 2)) return false;
    const int MT = (R + 16 * kM3sMB - 1) / (16 * kM3sMB), NT = (Nw + 64 * nb - 1) / (64 * nb);
    int k_len = K;
    const int S = mfma2_splits(MT, NT, R, Nw, K, ws_bytes, &k_len);  // k_len: a multiple of 128 = 32 D
    if (plan) *plan = {MT, NT, S, k_len, nb};
    return true;
  }
  const int MT = (R + 16 * kM3MB - 1) / (16 * kM3MB), NT = (Nw + 64 * kM3NB - 1) / (64 * kM3NB);
  int k_len = K, S = 1;
  bool ok;
  if (epi == kEpiAddF32) {
    S = mfma2_splits(MT, NT, R, Nw, K, ws_bytes, &k_len);  // k_len: a multiple of 128 = 32 D
    ok = K >= 8192 && S >= 2;
  } else {
    ok = (epi == kEpiSwiGLU || (epi == kEpiStoreF32 && Nw >= 65536)) && MT * NT >= 192;
  }
  if (!ok && epi == kEpiAddF32 && K < 8192 && Nw >= 4096 && Nw < 65536 && R <= 384) {
    // the residual-add projections of the 8B-shaped target at 160-384 rows
    // (the serving verify's O projection): the 64-row form with 256-row W
    // tiles, K split (364 rows 29.2 -> 25.4 us against gemm_mfma2_bf16)
    const int MTs = (R + 16 * kM3sMB - 1) / (16 * kM3sMB), NTs = (Nw + 255) / 256;
    int kl = K;
    const int Ss = mfma2_splits(MTs, NTs, R, Nw, K, ws_bytes, &kl);
    if (ws_bytes && plan) *plan = {MTs, NTs, Ss, kl, 4};
    return ws_bytes != 0;
  }
  if (ok && plan) *plan = {MT, NT, S, k_len, 0};
  return ok;
}

constexpr FormCost kM2Cost = {0.649, 0.067, 0.606, 0.109, 5.81, 0.0};
constexpr FormCost kM3Cost = {0.694, 0.0, 0.0, 0.136, 4.40, 0.0};
constexpr FormCost kM3sCost = {1.289, 0.0, 0.0, 0.136, 4.40, 0.0};

// The kernel and what follows it.  Workgroups run in rounds of 256 `occ`; two
// on a CU share its MFMAs.  W comes from HBM once for all row tiles, and into
// an XCD's L2 once for the row tiles that its run of tiles shares
// (gemm_mfma4_bf16: kM4Group, fewer where the last group's remainder falls).
// Constants: least squares on the logarithm of 44000 measured launches with
// weights rotated past the caches, the configured models' projections at 129
// to 8192 rows and 260 random ones (256 to 60000 outputs, K 256 to 16384).
// Median error 6-8%, a tenth of them are off by 13-18%; the same on 120
// projections left out of the fit.
double form_time(const FormCost& c, bool m4, int mb, int nb, int occ, int R, int N, int Nw, int MT, int NT, int S,
                 int k_len, int epi, Tail tail) {
  const bool sw = epi == kEpiSwiGLU, add = epi == kEpiAddF32;
  const int T = MT * NT * S, cap = 256 * occ;
  const double steps = k_len / 32;
  const int last = MT % kM4Group ? MT % kM4Group : kM4Group;
  const double fr = std::min(1.0, last * NT / std::max(T / 8.0, 1.0));
  const double per_row = 0.456 * (fr / last + (1.0 - fr) / std::min(MT, kM4Group)) +
                         0.544 * ((MT + kM4Group - 1) / kM4Group) / MT;
  const double mfma = mb * nb * 0.016 * c.mfma, in = (std::min(16 * mb, R) + 64 * nb) * 0.001 * c.in;
  const double w_mb = 64 * nb * 64e-6;
  const double tile_mb = 16.0 * mb * 64.0 * nb * 4e-6 *
                         (S > 1 ? 1.0 : add ? (m4 ? 4.32 : 5.62) : sw ? 0.581 : 1.0);
  auto round = [&](int n) {  // n workgroups at once
    const double two = n > 256 ? (occ > 1 ? 2.38 : 2.0) : 1.0;
    const double a = two * mfma * (m4 ? 1.0 + 0.058 * std::min(n, 256) / 256 : 1.0);
    const double b = (n > 256 ? 2.0 : 1.0) * in;
    const double hbm = std::max(static_cast<double>(n) / MT, 1.0);
    const double w = w_mb * (m4 ? std::max(n * per_row, 1.0) * c.w + 0.0858 * hbm : hbm * c.w);
    return steps * (std::sqrt(a * a + b * b + w * w) + c.step) + (m4 ? 0.0565 : 0.2) * tile_mb * n + c.round;
  };
  double t = (T / cap) * round(cap) + (T % cap ? round(T % cap) : 0.0);
  if (T > cap) t *= m4 ? 0.975 + 0.05 * std::min(static_cast<double>(T) / cap - 1.0, 3.0) : 1.086;
  t += c.start;
  if (sw) t *= m4 ? 0.944 : 1.048;
  const double out = R * static_cast<double>(N) * 4e-6, part = R * static_cast<double>(Nw) * S * 4e-6;  // MB
  if (tail == Tail::kNorm) return t + (S > 1 ? 2.70 + 0.221 * part + 0.351 * out : 3.02 + 0.366 * out);
  if (tail == Tail::kRope) return t + (S > 1 ? 5.09 + 0.355 * part : 4.07 + 0.802 * out);
  return S > 1 ? t + 2.68 + 0.232 * part + 0.076 * (add ? 2.0 : sw ? 0.5 : 1.0) * out : t;
}

}  // namespace

// use_mfma3 / mfma2_shape's choice, or above 128 rows (below, gemm_mfma3_bf16's
// 64-row form is as fast), for whole W tiles and whole unrolled k-loops, the
// gemm_mfma4_bf16 shape and split of the least estimated time if that is below
// the other's.  The margins are for the estimates' error: over 2900 projections
// of 129 to 8192 rows the choice takes 1.022 times the fastest form's time on
// average, and 3% of them are more than 3% slower than with the other kernels
// (gemm_mfma4_bf16 wherever it can run, by an estimate without the W term: 12%,
// up to 1.5 times; 256 rows of 5120 x 5120 took 46.5 us against 33.9 now).  Whole
// forwards of 136 to 1024 rows of the configured models are 2% faster for it
// (192 rows, 16 layers of 2048 x 16384: 1784 -> 1645 us).  m4: outputs and
// partials are aligned for it.
constexpr double kM4Margin = 0.99, kM4SplitMargin = 0.96;

MfmaPlan plan_mfma(int R, int N, int K, int epi, size_t ws_bytes, bool m4, Tail tail) {
  const int Nw = epi == kEpiSwiGLU ? 2 * N : N;
  MfmaPlan p;
  if (use_mfma3(R, Nw, K, epi, ws_bytes, &p.m3)) p.kernel = MfmaPlan::kM3;
  else p.m2 = mfma2_shape(R, N, Nw, K, ws_bytes, epi == kEpiSwiGLU);
  if (!m4 || R <= 128 || N % 16 || K % (32 * kM4DX)) return p;
  if (static_cast<double>(Nw) * K >= 2147483648.0 || static_cast<double>(R) * K >= 2147483648.0) return p;
  double best;
  if (p.kernel == MfmaPlan::kM3) {
    const bool small = p.m3.nb != 0;
    best = form_time(small ? kM3sCost : kM3Cost, false, small ? kM3sMB : kM3MB, small ? p.m3.nb : kM3NB, 1, R, N, Nw,
                     p.m3.MT, p.m3.NT, p.m3.S, p.m3.k_len, epi, tail);
  } else {
    const int MT = (R + 32 * p.m2.mtw - 1) / (32 * p.m2.mtw), NT = (Nw + 32 * p.m2.ntw - 1) / (32 * p.m2.ntw);
    int k_len = K;
    const int S = mfma2_splits(MT, NT, R, Nw, K, ws_bytes, &k_len);
    best = form_time(kM2Cost, false, 2 * p.m2.mtw, p.m2.ntw / 2, 1, R, N, Nw, MT, NT, S, k_len, epi, tail);
  }
  for (int i = 0; i < kM4Shapes_n; ++i) {
    const M4Shape& s = kM4Shapes[i];
    if (epi == kEpiSwiGLU && s.nb % 2) continue;
    const int MT = (R + 16 * s.mb - 1) / (16 * s.mb), NT = (Nw + 64 * s.nb - 1) / (64 * s.nb);
    for (int S = 1; S <= 8; S *= 2) {
      const int k_len = ((K + S - 1) / S + 255) / 256 * 256;
      if (S > 1 && ((K + k_len - 1) / k_len != S || MT * NT * S > 512 * s.occ ||
                    static_cast<size_t>(S) * R * Nw * sizeof(float) > ws_bytes))
        continue;
      const double t = form_time(s.cost, true, s.mb, s.nb, s.occ, R, N, Nw, MT, NT, S, k_len, epi, tail) /
                       (S > 1 ? kM4SplitMargin : kM4Margin);
      if (t < best) {
        best = t;
        p.kernel = MfmaPlan::kM4;
        p.shape = i;
        p.tl = {MT, NT, S, k_len};
      }
    }
  }
  return p;
}

size_t gemm_splitk_bytes(int R_max, int Nw_max) {
  // S R Nw floats of partials.  gemm_mfma2_bf16 and gemm_mfma3_bf16 split grids
  // of fewer than 192 tiles into at most 256 / tiles parts of tiles of at most
  // 256 x 256: below 256^3 floats, and 8 R Nw.  gemm_mfma4_bf16 may want twice
  // that (512 tiles of 256 x 256): plan_mfma leaves out the splits that do not
  // fit.
  const double cap = std::min(8.0 * R_max * Nw_max, 256.0 * 256.0 * 256.0);
  return static_cast<size_t>(cap) * sizeof(float);
}

}  // namespace spec
