// Paged causal grouped-query attention on gfx950.
//
// Row r of sequence s sits at absolute position pos_r and attends keys
// 0..pos_r of its own cache (the verify window's K/V are written before this
// kernel runs, so drafts see each other causally).  Query head h reads kv head
// h / (Hq / Hkv).  Scale 1/sqrt(hd).
//
// KV pages hold 16 tokens per (page, kv head) block, in the operand order of
// kv_layout.h for bf16 (K as [16][hd] and V transposed as [hd][16] for fp32).
// The bf16 kernel gives each workgroup of W waves one (rows of one sequence,
// kv head, key range) work item and runs both products on MFMA:
//   S^T = K Q^T : A = 16 keys x 32 dims of K, B = 32 dims x 16 query vectors.
//   O^T = V^T P^T: A = 16 dims x 32 keys of V^T, B = P^T.
// Keys inside each 32-key chunk are permuted (A row i of key tile h reads key
// 8 (i / 4) + 4 h + i % 4) so that the S^T accumulators a lane ends up with are
// exactly the 8 consecutive keys it must supply as the P^T operand, and the
// softmax statistics of query vector (l % 16) stay lane-local: no shuffles of
// P, no LDS in the loop.  With the page layout of kv_layout.h every K and V^T
// operand load of a wave reads two contiguous 512-byte runs.  Long contexts
// are split into key ranges (multiples of 32) whose unnormalised partials a
// combine kernel merges.

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <type_traits>

#include "attention.h"
#include "common.h"

namespace spec {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kAttnStagedPages = 256;  // page ids of one work item kept in LDS (4096 keys)

__device__ __forceinline__ uint32_t mask_pair(uint32_t w, int valid) {
  // keep the first `valid` (0, 1, 2) bf16 halves of a 32-bit word
  return valid >= 2 ? w : (valid == 1 ? (w & 0xFFFFu) : 0u);
}

// W waves per workgroup share one work item: wave w takes the 32-key chunks
// w, w + W, ... of the item's key range, and the waves' softmax states are
// merged through LDS at the end (exact rescaling by exp2(m_w - m)).
template <int HD, int NT, int W, bool TREE>
__device__ __forceinline__ void attn_bf16_body(const AttnArgs& a, const AttnItem* __restrict__ items) {
  constexpr int DS = HD / 32;   // MFMA k-steps over the head dim
  constexpr int DT = HD / 16;   // 16-dim output tiles
  // the kv heads of an item run side by side: their blocks of a page are one
  // run of memory (loads alone, 64-sequence verify: 72-87 us with the items
  // first, depending on the split, 71-73 us with the heads first)
  const int gkv = blockIdx.x % a.Hkv;
  const AttnItem it = items[blockIdx.x / a.Hkv];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane >> 4, l16 = lane & 15;
  const int G = a.Hq / a.Hkv;
  const int M = it.nrows * G;
  const bf16_t* q = static_cast<const bf16_t*>(a.q);
  const bf16_t* kp = static_cast<const bf16_t*>(a.kpool);
  const bf16_t* vp = static_cast<const bf16_t*>(a.vpool);
  const int32_t* pt = a.page_table + static_cast<size_t>(it.seq) * a.max_pages;
  // the item's page ids, staged once in LDS so that no chunk waits on a
  // page-table load before its K / V loads can go out (items spanning more
  // pages than the stage holds read the table directly)
  __shared__ int32_t s_pt[kAttnStagedPages];
  const int p0 = it.t0 >> 4;
  const int np = it.t1 > it.t0 ? ((it.t1 - 1) >> 4) - p0 + 1 : 0;
  const bool staged = np <= kAttnStagedPages;
  if (staged)
    for (int i = threadIdx.x; i < np; i += kWave * W) s_pt[i] = pt[p0 + i];
  __syncthreads();

  uint4 qf[NT][DS];
  int vpos[NT];
  uint32_t tmask[NT];
  bool vval[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int m = 16 * nt + l16;
    vval[nt] = m < M;
    const int mm = vval[nt] ? m : 0;
    if constexpr (TREE) {
      // vpos: the last index every row sees; beyond it the tree's bits
      vpos[nt] = a.tree_base[it.row0 + mm / G];
      tmask[nt] = a.tree_mask[it.row0 + mm / G];
    } else {
      vpos[nt] = it.pos0 + mm / G;
      tmask[nt] = 0u;
    }
    const bf16_t* base =
        q + (static_cast<size_t>(it.row0 + mm / G) * a.Hq + gkv * G + mm % G) * HD + g * 8;
#pragma unroll
    for (int s = 0; s < DS; ++s)
      qf[nt][s] = vval[nt] ? reinterpret_cast<const uint4*>(base)[4 * s] : make_uint4(0, 0, 0, 0);
  }
  const float scale = kLog2e / sqrtf(static_cast<float>(HD));
  // every row of the item sees the keys up to here
  const int pos_lo = TREE ? a.tree_base[it.row0] : it.pos0;
  float mrun[NT], lrun[NT];
  f32x4 acc[DT][NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    mrun[nt] = -INFINITY;
    lrun[nt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // The wave's chunks.  One K and one V^T buffer: the next chunk's K is loaded
  // once this chunk's scores are computed, its V^T once this chunk's output
  // update is done (loads are unconditional, clamped past the end, so that the
  // compiler's waits stay exact), which keeps 16 KB of a head dim of 128 in
  // flight per wave.  The page ids come from LDS or from the table in two
  // instances of the loop: a choice per load made the compiler fetch them by
  // flat loads, whose waits drained every load in flight twice a chunk (the
  // 64-sequence verify ran at 4.6 TB/s).
  auto walk = [&](auto from_lds) {
    auto page = [&](int t) {
      if constexpr (decltype(from_lds)::value) return s_pt[(t >> 4) - p0];
      else return pt[t >> 4];
    };
    // K and V^T operands of one 32-key chunk (keys past t1 are clamped to a
    // valid address; their scores are masked and their V entries zeroed)
    auto load_k = [&](int c0, uint4 (&kf)[2][DS]) {
      // lanes 0-7 / 8-15 of a group read the chunk's first / second page:
      // unit ((s * 2 + hh) * 4 + g) * 8 + l16 % 8 of the page's K block holds
      // dims 32 s + 8 g .. of key 8 (l16 / 4) + 4 hh + l16 % 4 (kv_layout.h)
      const int tk = min(c0 + 16 * (l16 >> 3), it.t1 - 1);
      const uint4* kb = reinterpret_cast<const uint4*>(kp + static_cast<size_t>(page(tk) * a.Hkv + gkv) * 16 * HD);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int s = 0; s < DS; ++s) kf[hh][s] = ld_stream(kb + ((s * 2 + hh) * 4 + g) * 8 + (l16 & 7));
    };
    auto load_v = [&](int c0, uint4 (&vf)[DT]) {
      // V^T: unit (dt * 2 + g % 2) * 16 + l16 holds keys 8 (g % 2) .. + 7 of
      // dim 16 dt + l16 of page (c0 + 8 g) / 16
      const int tvc = min(c0 + 8 * g, it.t1 - 1);
      const uint4* vb = reinterpret_cast<const uint4*>(vp + static_cast<size_t>(page(tvc) * a.Hkv + gkv) * HD * 16);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vf[dt] = ld_stream(vb + (dt * 2 + (g & 1)) * 16 + l16);
    };
    uint4 kf[2][DS], vf[DT];
    const int cfirst = it.t0 + 32 * wave;
    if (cfirst < it.t1) {
      load_k(cfirst, kf);
      load_v(cfirst, vf);
    }
    for (int c0 = cfirst; c0 < it.t1; c0 += 32 * W) {
      const int cn = min(c0 + 32 * W, it.t1 - 1);
      // every key inside the item and seen by every row: no masks
      const bool full = c0 + 32 <= it.t1 && c0 + 31 <= pos_lo;
      f32x4 sc[NT][2];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < DS; ++s) {
          s0 = mfma16x16x32(kf[0][s], qf[nt][s], s0);
          s1 = mfma16x16x32(kf[1][s], qf[nt][s], s1);
        }
        sc[nt][0] = s0;
        sc[nt][1] = s1;
      }
      load_k(cn, kf);
      // raw scores, -inf where masked; the running maxima; the smallest exponent
      float raw[NT][8], mneg[NT];
      bool low = false;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
        for (int j = 0; j < 8; ++j) raw[nt][j] = (j < 4) ? sc[nt][0][j] : sc[nt][1][j - 4];
        if (!full) {
          asm volatile("");  // keeps the masks a branch
          // (selects of scalars, not `if (!ok) sc[nt][..] = -INFINITY`: compiled
          // from && and || that put the score back in masked lanes)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int t = c0 + 8 * g + j;
            bool ok = vval[nt] & (t < it.t1);
            if constexpr (TREE) {
              const int rel = t - vpos[nt];
              ok = ok & ((rel <= 0) | ((rel <= 32) & (((tmask[nt] >> ((rel - 1) & 31)) & 1u) != 0)));
            } else {
              ok = ok & (t <= vpos[nt]);
            }
            raw[nt][j] = ok ? raw[nt][j] : -INFINITY;
          }
        }
        float mx = raw[nt][0], mn = mx;
#pragma unroll
        for (int j = 1; j < 8; ++j) {
          mx = fmaxf(mx, raw[nt][j]);
          mn = fminf(mn, raw[nt][j]);
        }
        mx *= scale;  // base-2 logit (scale > 0)
        // a new maximum: the same in every lane of a query vector
        if (__any(mx > mrun[nt])) {
          mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
          mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
          const bool grow = mx > mrun[nt];
          const float alpha = grow ? ((mrun[nt] == -INFINITY) ? 0.f : exp2f(mrun[nt] - mx)) : 1.f;
          if (grow) mrun[nt] = mx;
          lrun[nt] *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) acc[dt][nt] *= alpha;
        }
        mneg[nt] = (mrun[nt] == -INFINITY) ? -INFINITY : -mrun[nt];
        low |= fmaf(mn, scale, mneg[nt]) < -126.f;
      }
      uint4 pf[NT];
      auto probabilities = [&](auto exp2) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          float p[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) p[j] = exp2(fmaf(raw[nt][j], scale, mneg[nt]));
          float ps = 0.f;
#pragma unroll
          for (int j = 0; j < 8; ++j) ps += p[j];
          lrun[nt] += ps;
          pf[nt] = make_uint4(cvt_pk_bf16(p[0], p[1]), cvt_pk_bf16(p[2], p[3]), cvt_pk_bf16(p[4], p[5]),
                              cvt_pk_bf16(p[6], p[7]));
        }
      };
      // v_exp_f32 flushes results below 2^-126 to 0, bf16 probabilities go down
      // to 2^-133: it serves where no exponent is that low (one test for all
      // tiles; 64-sequence verify 91 us with the test, without and with exp2f
      // everywhere; 64 x 16 rows, head dim 64, 4000 keys 140, 131 and 151)
      if (__any(low)) probabilities([](float x) { return exp2f(x); });
      else probabilities([](float x) { return __builtin_amdgcn_exp2f(x); });
      if (c0 + 32 > it.t1) {  // keys past the end hold anything, and 0 x NaN is not 0
        asm volatile("");
        const int nvalid = min(max(it.t1 - (c0 + 8 * g), 0), 8);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          vf[dt].x = mask_pair(vf[dt].x, nvalid);
          vf[dt].y = mask_pair(vf[dt].y, nvalid - 2);
          vf[dt].z = mask_pair(vf[dt].z, nvalid - 4);
          vf[dt].w = mask_pair(vf[dt].w, nvalid - 6);
        }
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[dt][nt] = mfma16x16x32(vf[dt], pf[nt], acc[dt][nt]);
      load_v(cn, vf);
    }
  };
  if (staged) walk(std::true_type{});
  else walk(std::false_type{});

  float ltot[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float lt = lrun[nt];
    lt += __shfl_xor(lt, 16, kWave);
    lt += __shfl_xor(lt, 32, kWave);
    ltot[nt] = lt;
  }
  if (W > 1) {
    // waves 1..W-1 hand their state to wave 0 (same lane layout in every wave)
    __shared__ float s_acc[W > 1 ? W - 1 : 1][NT][DT][4][kWave];
    __shared__ float s_ml[W > 1 ? W - 1 : 1][NT][2][kWave];
    if (wave > 0) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        s_ml[wave - 1][nt][0][lane] = mrun[nt];
        s_ml[wave - 1][nt][1][lane] = ltot[nt];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 4; ++r) s_acc[wave - 1][nt][dt][r][lane] = acc[dt][nt][r];
      }
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      float mm = mrun[nt];
      for (int w = 0; w < W - 1; ++w) mm = fmaxf(mm, s_ml[w][nt][0][lane]);
      if (mm == -INFINITY) continue;  // no key of the item for this query vector
      const float e0 = (mrun[nt] == -INFINITY) ? 0.f : exp2f(mrun[nt] - mm);
      float lt = ltot[nt] * e0;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt][nt] *= e0;
      for (int w = 0; w < W - 1; ++w) {
        const float mw = s_ml[w][nt][0][lane];
        const float ew = (mw == -INFINITY) ? 0.f : exp2f(mw - mm);
        lt += ew * s_ml[w][nt][1][lane];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[dt][nt][r] += ew * s_acc[w][nt][dt][r][lane];
      }
      mrun[nt] = mm;
      ltot[nt] = lt;
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float lt = ltot[nt];
    const int m = 16 * nt + l16;
    if (m >= M) continue;
    if (it.part < 0) {
      const float inv = (lt > 0.f) ? 1.f / lt : 0.f;
      bf16_t* o = static_cast<bf16_t*>(a.out) +
                  (static_cast<size_t>(it.row0 + m / G) * a.Hq + gkv * G + m % G) * HD;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const f32x4 v = acc[dt][nt];
        *reinterpret_cast<uint2*>(o + 16 * dt + 4 * g) =
            make_uint2(pack_bf16x2(v[0] * inv, v[1] * inv), pack_bf16x2(v[2] * inv, v[3] * inv));
      }
    } else {
      const size_t pm = static_cast<size_t>(it.part * a.Hkv + gkv) * 64 + m;
      float* po = a.part_o + pm * HD;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        *reinterpret_cast<float4*>(po + 16 * dt + 4 * g) =
            make_float4(acc[dt][nt][0], acc[dt][nt][1], acc[dt][nt][2], acc[dt][nt][3]);
      if (g == 0) {
        a.part_ml[pm * 2] = mrun[nt];
        a.part_ml[pm * 2 + 1] = lt;
      }
    }
  }
}

// One workgroup per (group, kv head, 4 query vectors), one thread per (query
// vector, DPT consecutive head dims: DPT = 4 (float4 loads of the partial
// outputs) for head dim 128, 1 for head dim 64, as measured).  Up
// to kCombineOnePass parts: every part's (max, sum) and output vector is
// loaded before the first is used (one round trip), then the maximum and the
// weighted sums.  More parts: two passes (maximum, then weighted sums), each
// issuing batches of 8 independent loads.  Both sum the parts in index order,
// per element as a one-element-per-thread combine would.
constexpr int kCombineQv = 4;
constexpr int kCombineOnePass = 32;

template <int DPT>
struct CombVec;
template <>
struct CombVec<1> {
  float v[1];
  __device__ __forceinline__ void load(const float* p) { v[0] = *p; }
};
template <>
struct CombVec<4> {
  float v[4];
  __device__ __forceinline__ void load(const float* p) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
};

template <int HD, int NT, int W>
__global__ __launch_bounds__(64 * W, NT <= 2 ? 2 : 1) void attn_bf16_kernel(AttnArgs a, const AttnItem* __restrict__ items) {
  attn_bf16_body<HD, NT, W, false>(a, items);
}

// The same with the rows' tree masks (tree verification).
template <int HD, int NT, int W>
__global__ __launch_bounds__(64 * W, NT <= 2 ? 2 : 1) void attn_tree_bf16_kernel(AttnArgs a,
                                                                                  const AttnItem* __restrict__ items) {
  attn_bf16_body<HD, NT, W, true>(a, items);
}

// ---------------------------------------------------------------------------
// Causal prefill: long runs of consecutive rows of one sequence.  One
// workgroup of 8 waves (two per SIMD) per (block of 256 / G rows, kv head):
// its 256 query vectors (rows x the G query heads of the kv head) share every
// K / V load.  The keys 0 .. last row's position are brought into LDS 64 at a
// time (four pages of K and of V, three stage buffers) by direct-to-LDS loads
// of whole page blocks, and each wave runs both products for its own 32 query
// vectors (2 tiles) from there, with the key permutation and lane-local
// softmax of attn_bf16_body.  Each wave sees every key of its rows, so it
// normalises its own output: no key splits, no combine.
// A 32-key chunk is a matrix phase (its scores, the output update of the chunk
// before) and a vector phase (its softmax), a barrier after each, and waves
// 4..7 run one phase behind waves 0..3, with which they share the SIMDs: one
// of a SIMD's two waves multiplies while the other takes its exponentials.
// Measured by cycle counters: a phase pair costs about what the SIMD's MFMAs
// (512 cycles) and vector instructions (560) add up to, so the softmax is kept
// short: 8192 rows (32q / 8kv, head dim 128) 559 -> 490 us (970 -> 1120
// TFLOP/s), 2048 rows 89 -> 69 us, head dim 64 at 4096 rows 127 -> 114 us.
// That start and the last output update cost about 1 us, so up to
// kPrefillShortKeys keys a wave takes its chunks one after another with one
// barrier per stage (SHORT): 64 / 250 / 300 / 380 keys, 8q / 8kv, head dim 128,
// 6.8 / 14.6 / 15.5 / 16.3 us by phases, 6.1 / 13.0 / 14.1 / 15.2 in turn; from
// 500 keys on the phases are as fast or faster.
// The running maximum of a query vector is raised only when a score exceeds
// it by more than 2^8 (scores are base-2 logits): each lane compares its own
// 8 scores against it, and only when some lane of the wave finds a larger
// one does the wave take the cross-lane maximum and rescale its output
// accumulators.  Probabilities stay below 2^8 in between; the shared maximum
// is the same in every lane of a query vector, so the products stay exact.
// Chunks entirely at or below every row of a wave skip the causal mask.
constexpr float kPrefillRescaleLog2 = 8.f;
constexpr int kPrefillStagedPages = 1024;  // page ids kept in LDS (16384 keys)

template <int HD, bool SHORT>
__device__ __forceinline__ void attn_prefill_body(const AttnArgs& a, const AttnItem* __restrict__ items) {
  constexpr int DS = HD / 32;    // MFMA k-steps over the head dim
  constexpr int DT = HD / 16;    // 16-dim output tiles
  constexpr int NT = 2;          // 16-vector query tiles per wave
  constexpr int NW = 8;          // waves
  constexpr int BU = 2 * HD;     // 16-byte units of one (page, kv head) block
  constexpr int SU = 4 * BU;     // units of K (and of V) per 64-key stage
  constexpr int NB = 3;          // stage buffers
  constexpr int LPW = 2 * SU / (64 * NW);  // direct-to-LDS loads per wave per stage
  __shared__ uint4 sk[NB][SU], sv[NB][SU];
  __shared__ int32_t s_pt[kPrefillStagedPages];
  const int gkv = blockIdx.x % a.Hkv;
  const AttnItem it = items[blockIdx.x / a.Hkv];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform: load bases in SGPRs
  const int g = lane >> 4, l16 = lane & 15;
  const int G = a.Hq / a.Hkv;
  const bf16_t* q = static_cast<const bf16_t*>(a.q);
  const bf16_t* kp = static_cast<const bf16_t*>(a.kpool);
  const bf16_t* vp = static_cast<const bf16_t*>(a.vpool);
  const int32_t* pt = a.page_table + static_cast<size_t>(it.seq) * a.max_pages;
  const int t1 = it.t1;                 // keys 0 .. t1 - 1 (t0 = 0)
  const int np = (t1 + 15) >> 4;
  const int ns = (t1 + 63) >> 6;        // stages
  // (the planner keeps t1 <= 16 kPrefillStagedPages)
  for (int i = threadIdx.x; i < np; i += 64 * NW) s_pt[i] = pt[i];
  __syncthreads();

  // stage j (keys 64 j ..) into buffer b: wave w moves one page block, K of
  // page w of the stage for w < 4, V of page w - 4 after (its LPW loads of
  // 64 units each); pages past the sequence's last clamped to it (those keys
  // are masked)
  static_assert(LPW * 64 == BU && NW == 8, "one page block per wave and stage");
  const bool wv = wave >= 4;
  const int wpg = wave & 3;
  auto page_of = [&](int j) { return s_pt[min(4 * j + wpg, np - 1)]; };
  auto issue = [&](int page_id, int b) {
    const int page = __builtin_amdgcn_readfirstlane(page_id);
    const bf16_t* blk = (wv ? vp : kp) + static_cast<size_t>(page * a.Hkv + gkv) * 16 * HD;
    const uint32_t dst = lds_addr(wv ? &sv[b][wpg * BU] : &sk[b][wpg * BU]);
#pragma unroll
    for (int i = 0; i < LPW; ++i) load_lds16(blk, (i * 64 + lane) * 16, dst + i * 1024);
  };

  uint4 qf[NT][DS];
  bool vval[NT];
  int vpos[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int m = 32 * wave + 16 * nt + l16;
    vval[nt] = m / G < it.nrows;
    const int mm = vval[nt] ? m : 0;
    vpos[nt] = it.pos0 + mm / G;
    const bf16_t* base = q + (static_cast<size_t>(it.row0 + mm / G) * a.Hq + gkv * G + mm % G) * HD + g * 8;
#pragma unroll
    for (int s = 0; s < DS; ++s)
      qf[nt][s] = vval[nt] ? reinterpret_cast<const uint4*>(base)[4 * s] : make_uint4(0, 0, 0, 0);
  }
  // the last key each query vector sees (-1: none, a padding vector)
  int klim[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) klim[nt] = vval[nt] ? min(vpos[nt], t1 - 1) : -1;
  // the wave's rows: positions pos_lo .. pos_hi
  const int pos_lo = it.pos0 + (32 * wave) / G;
  const int pos_hi = it.pos0 + min((32 * wave + 31) / G, it.nrows - 1);
  const float scale = kLog2e / sqrtf(static_cast<float>(HD));
  // minus the running maximum (base-2 logits; -inf: no key yet, every p is 0),
  // the raw score above which it is raised, two partial sums of p
  float mneg[NT], mlim[NT], lrun[NT][2];
  f32x4 acc[DT][NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    mneg[nt] = mlim[nt] = -INFINITY;
    lrun[nt][0] = lrun[nt][1] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // K and V^T operands of 32-key chunk h of buffer b, read from LDS
  uint4 kf[2][DS], vf[DT];
  auto read_k = [&](int b, int h) {
    const uint4* kb = &sk[b][(2 * h + (l16 >> 3)) * BU];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int s = 0; s < DS; ++s) kf[hh][s] = kb[((s * 2 + hh) * 4 + g) * 8 + (l16 & 7)];
  };
  // (quarter q of V^T's tiles)
  auto read_v = [&](int b, int h, int q) {
    const uint4* vb = &sv[b][(2 * h + (g >> 1)) * BU];
#pragma unroll
    for (int dt = q * DT / 4; dt < (q + 1) * DT / 4; ++dt) vf[dt] = vb[(dt * 2 + (g & 1)) * 16 + l16];
  };
  f32x4 sc[NT][2];
  uint4 pf[NT];
  // scores of the chunk in kf
  auto scores = [&] {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) sc[nt][0] = sc[nt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DS; ++s)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) sc[nt][hh] = mfma16x16x32(kf[hh][s], qf[nt][s], sc[nt][hh]);
  };
  // output update with the chunk of keys c0 .. in vf and its probabilities in pf
  auto output = [&](int c0) {
    if (c0 + 32 > t1) {
      // keys past the sequence hold stale or uninitialised V (their
      // probabilities are 0, but 0 x NaN is not)
      asm volatile("");
      const int nvalid = min(max(t1 - (c0 + 8 * g), 0), 8);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        vf[dt].x = mask_pair(vf[dt].x, nvalid);
        vf[dt].y = mask_pair(vf[dt].y, nvalid - 2);
        vf[dt].z = mask_pair(vf[dt].z, nvalid - 4);
        vf[dt].w = mask_pair(vf[dt].w, nvalid - 6);
      }
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[dt][nt] = mfma16x16x32(vf[dt], pf[nt], acc[dt][nt]);
  };
  // probabilities of the chunk of keys c0 .. from its scores, with the reads
  // of the chunk's V^T (chunk h of buffer b) between them: issued together
  // they held the wave at the LDS pipe before its arithmetic could start.
  // Both query tiles go through each branch together: taken branches cost more
  // than the few instructions they skip.
  auto softmax = [&](int c0, int b, int h) {
    read_v(b, h, 0);
    read_v(b, h, 1);
    // some key above a row of the wave or past the sequence
    if (c0 + 31 > pos_lo || c0 + 31 >= t1) {
      asm volatile("");  // keeps the mask a branch around diagonal chunks (not selects everywhere)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (c0 + 8 * g + j > klim[nt]) sc[nt][j / 4][j % 4] = -INFINITY;
    }
    float mx[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      mx[nt] = sc[nt][0][0];
#pragma unroll
      for (int j = 1; j < 8; ++j) mx[nt] = fmaxf(mx[nt], sc[nt][j / 4][j % 4]);
    }
    static_assert(NT == 2, "one test for both tiles");
    if (__any(mx[0] > mlim[0] || mx[1] > mlim[1])) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        // the query vector's maximum over the chunk, from all lanes holding it
        float m = mx[nt];
        m = fmaxf(m, __shfl_xor(m, 16, kWave));
        m = fmaxf(m, __shfl_xor(m, 32, kWave));
        if (m > mlim[nt]) {
          const float mb = m * scale;  // base-2 logit (scale > 0)
          const float alpha = mneg[nt] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(-mneg[nt] - mb);
          mneg[nt] = -mb;
          mlim[nt] = m + kPrefillRescaleLog2 / scale;
#pragma unroll
          for (int i = 0; i < 2; ++i) lrun[nt][i] *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) acc[dt][nt] *= alpha;
        }
      }
    }
    read_v(b, h, 2);
    read_v(b, h, 3);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      // p = 2^(raw scale - m): one FMA per score
      float p[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) p[j] = __builtin_amdgcn_exp2f(fmaf(sc[nt][j / 4][j % 4], scale, mneg[nt]));
#pragma unroll
      for (int j = 0; j < 8; ++j) lrun[nt][j % 2] += p[j];
      pf[nt] = make_uint4(cvt_pk_bf16(p[0], p[1]), cvt_pk_bf16(p[2], p[3]), cvt_pk_bf16(p[4], p[5]),
                          cvt_pk_bf16(p[6], p[7]));
    }
  };
  auto phase_end = [&] {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  };

  issue(page_of(0), 0);
  if (ns > 1) issue(page_of(1), 1);
  if constexpr (SHORT) {
    for (int j = 0; j < ns; ++j) {
      // stage j has landed (stage j + 1 may be in flight), every wave is done
      // with stage j - 1, whose buffer takes stage j + 2
      if (j + 1 < ns) {
        SPEC_WAIT_VM_LDS(LPW);
      } else {
        SPEC_WAIT_VM_LDS(0);
      }
      phase_end();
      if (j + 2 < ns) issue(page_of(j + 2), (j + 2) % NB);
      const int b = j % NB;
      read_k(b, 0);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c0 = 64 * j + 32 * h;
        if (c0 > pos_hi) break;  // above every row of this wave
        scores();
        if (h == 0) read_k(b, 1);
        softmax(c0, b, h);
        output(c0);
      }
    }
  } else {
    if (ns > 1) {
      SPEC_WAIT_VM_LDS(LPW);
    } else {
      SPEC_WAIT_VM_LDS(0);
    }
    int page_next = page_of(2);
    phase_end();  // stage 0 has landed
    read_k(0, 0);
    if (wave >= 4) phase_end();  // waves 4..7 run one phase behind
    for (int j = 0; j < ns; ++j) {
      const int b = j % NB, bn = (j + 1) % NB;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c0 = 64 * j + 32 * h;
        // matrix phase (chunks above every row of this wave are left out); the
        // next chunk's K as soon as the scores have taken this one's
        if (c0 <= pos_hi) scores();
        if (h == 0) read_k(b, 1);
        else if (j + 1 < ns) read_k(bn, 0);
        if (c0 >= 32 && c0 - 32 <= pos_hi) output(c0 - 32);
        // stage j + 1 has landed before any wave reads it, a phase on
        if (h == 0) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        phase_end();
        // vector phase.  Every wave is past its reads of stage j - 1 (the last
        // were waited for before the barrier just passed), so its buffer takes
        // stage j + 2
        if (h == 0 && j + 2 < ns) issue(page_next, (j + 2) % NB);
        if (h == 1) page_next = page_of(j + 3);
        __builtin_amdgcn_s_setprio(1);  // (head dim 64: 2% faster)
        if (c0 <= pos_hi) softmax(c0, b, h);
        __builtin_amdgcn_s_setprio(0);
        SPEC_WAIT_VM_LDS(63);  // (LDS reads only)
        phase_end();
      }
    }
    if (64 * ns - 32 <= pos_hi) output(64 * ns - 32);
    if (wave < 4) phase_end();
  }

#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float lt = lrun[nt][0] + lrun[nt][1];
    lt += __shfl_xor(lt, 16, kWave);
    lt += __shfl_xor(lt, 32, kWave);
    const int m = 32 * wave + 16 * nt + l16;
    if (!vval[nt]) continue;
    const float inv = (lt > 0.f) ? 1.f / lt : 0.f;
    bf16_t* o = static_cast<bf16_t*>(a.out) + (static_cast<size_t>(it.row0 + m / G) * a.Hq + gkv * G + m % G) * HD;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4 v = acc[dt][nt];
      *reinterpret_cast<uint2*>(o + 16 * dt + 4 * g) =
          make_uint2(pack_bf16x2(v[0] * inv, v[1] * inv), pack_bf16x2(v[2] * inv, v[3] * inv));
    }
  }
}

template <int HD>
__global__ __launch_bounds__(512, 1) void attn_prefill_bf16_kernel(AttnArgs a, const AttnItem* __restrict__ items) {
  attn_prefill_body<HD, false>(a, items);
}
template <int HD>
__global__ __launch_bounds__(512, 1) void attn_prefill_short_bf16_kernel(AttnArgs a,
                                                                         const AttnItem* __restrict__ items) {
  attn_prefill_body<HD, true>(a, items);
}

template <int HD, int DPT>
__global__ __launch_bounds__(HD / DPT * kCombineQv) void attn_combine_kernel(AttnArgs a,
                                                                              const AttnGroup* __restrict__ groups) {
  constexpr int TQ = HD / DPT;  // threads per query vector
  const AttnGroup gr = groups[blockIdx.x];
  const int gkv = blockIdx.y;
  const int m = blockIdx.z * kCombineQv + static_cast<int>(threadIdx.x) / TQ;
  const int G = a.Hq / a.Hkv;
  if (m >= gr.nrows * G) return;
  const int d0 = DPT * (threadIdx.x % TQ);  // dims d0 .. d0 + DPT - 1
  const int n = gr.nparts;
  const size_t base = static_cast<size_t>(gr.part0 * a.Hkv + gkv) * 64 + m;
  const size_t stride = static_cast<size_t>(a.Hkv) * 64;
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml);
  float num[DPT];
#pragma unroll
  for (int i = 0; i < DPT; ++i) num[i] = 0.f;
  float den = 0.f;
  auto acc = [&](float w, const CombVec<DPT>& o, float l) {
#pragma unroll
    for (int i = 0; i < DPT; ++i) num[i] += w * o.v[i];
    den += w * l;
  };
  if (n <= kCombineOnePass) {
    float2 mlc[kCombineOnePass];
    CombVec<DPT> oc[kCombineOnePass];
#pragma unroll
    for (int j = 0; j < kCombineOnePass; ++j)
      if (j < n) {
        const size_t pm = base + j * stride;
        mlc[j] = ml[pm];
        oc[j].load(a.part_o + pm * HD + d0);
      }
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < kCombineOnePass; ++j)
      if (j < n) mx = fmaxf(mx, mlc[j].x);
    if (mx != -INFINITY) {
#pragma unroll
      for (int j = 0; j < kCombineOnePass; ++j)
        if (j < n) acc(mlc[j].x != -INFINITY ? exp2f(mlc[j].x - mx) : 0.f, oc[j], mlc[j].y);
    }
  } else {
    constexpr int B = 8;
    float mx = -INFINITY;
    for (int c0 = 0; c0 < n; c0 += B) {
      float mc[B];
#pragma unroll
      for (int j = 0; j < B; ++j) mc[j] = ml[base + min(c0 + j, n - 1) * stride].x;
#pragma unroll
      for (int j = 0; j < B; ++j) mx = fmaxf(mx, mc[j]);
    }
    if (mx != -INFINITY) {
      for (int c0 = 0; c0 < n; c0 += B) {
        float2 mc[B];
        CombVec<DPT> oc[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
          const size_t pm = base + min(c0 + j, n - 1) * stride;
          mc[j] = ml[pm];
          oc[j].load(a.part_o + pm * HD + d0);
        }
#pragma unroll
        for (int j = 0; j < B; ++j)
          if (c0 + j < n) acc(mc[j].x != -INFINITY ? exp2f(mc[j].x - mx) : 0.f, oc[j], mc[j].y);
      }
    }
  }
  const size_t o = (static_cast<size_t>(gr.row0 + m / G) * a.Hq + gkv * G + m % G) * HD + d0;
  const bool ok = den > 0.f;
  bf16_t* out = static_cast<bf16_t*>(a.out) + o;
  if constexpr (DPT == 4) {
    *reinterpret_cast<uint2*>(out) = make_uint2(pack_bf16x2(ok ? num[0] / den : 0.f, ok ? num[1] / den : 0.f),
                                                pack_bf16x2(ok ? num[2] / den : 0.f, ok ? num[3] / den : 0.f));
  } else {
    out[0] = f32_to_bf16(ok ? num[0] / den : 0.f);
  }
}

// fp32: one workgroup of 256 threads per (row, head), 256 keys at a time: a
// thread scores one key (its K row in 16-byte loads), then thread (dim, part)
// sums the probabilities times V^T over every (256 / HD)th page, 16 keys of
// one dim in four loads.  Every load of a step is independent, so a step is
// two round trips whatever the context: with one wave per (row, head) whose
// lanes walked their keys one after another, 5 rows over 128 keys took 38 us
// against 6 now.  Masked keys are skipped (their V may hold anything).
template <int HD>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a, const int32_t* __restrict__ row_seq,
                                                       const int32_t* __restrict__ row_pos) {
  constexpr int T = 256, NW = T / kWave, PARTS = T / HD;
  const int r = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const int wave = tid / kWave, lane = tid & (kWave - 1);
  const int G = a.Hq / a.Hkv, gkv = h / G;
  // causal by position, or the row's tree keys: 0..base and base + 1 + j for
  // the bits j of its mask
  const bool tree = a.tree_base != nullptr;
  const int base = tree ? a.tree_base[r] : row_pos[r];
  const uint32_t tm = tree ? a.tree_mask[r] : 0u;
  const int tlim = base + 1 + (tm ? 32 - __clz(static_cast<int>(tm)) : 0);
  const int32_t* pt = a.page_table + static_cast<size_t>(row_seq[r]) * a.max_pages;
  const float* kp = static_cast<const float*>(a.kpool);
  const float* vp = static_cast<const float*>(a.vpool);
  __shared__ f32x4 qs[HD / 4];
  __shared__ float sp[T];  // probabilities of the step's keys, -1 where masked
  __shared__ float wmax[NW], wsum[NW];
  __shared__ float part[PARTS][HD];
  const float* qv = static_cast<const float*>(a.q) + (static_cast<size_t>(r) * a.Hq + h) * HD;
  if (tid < HD) reinterpret_cast<float*>(qs)[tid] = qv[tid];
  __syncthreads();
  const float scale = 1.f / sqrtf(static_cast<float>(HD));
  const int d = tid % HD, pw = tid / HD;
  float m = -INFINITY, l = 0.f, o = 0.f;
  for (int c0 = 0; c0 < tlim; c0 += T) {
    const int t = c0 + tid;
    const bool ok = t < tlim && (t <= base || ((tm >> (t - base - 1)) & 1u));
    float s = -INFINITY;
    if (ok) {
      const f32x4_any* kr = reinterpret_cast<const f32x4_any*>(
          kp + (static_cast<size_t>(pt[t >> 4] * a.Hkv + gkv) * 16 + (t & 15)) * HD);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < HD / 4; ++i) {
        const f32x4 k = kr[i], q = qs[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(q[e], k[e], acc[e]);
      }
      s = ((acc[0] + acc[1]) + (acc[2] + acc[3])) * scale;
    }
    const float sm = wave_max(s);
    if (lane == 0) wmax[wave] = sm;
    __syncthreads();
    float mn = m;
#pragma unroll
    for (int w = 0; w < NW; ++w) mn = fmaxf(mn, wmax[w]);  // (key 0 is never masked: finite for finite scores)
    const float al = (m == -INFINITY) ? 0.f : expf(m - mn);
    const float p = ok ? expf(s - mn) : 0.f;
    sp[tid] = ok ? p : -1.f;
    const float ps = wave_sum(p);
    if (lane == 0) wsum[wave] = ps;
    m = mn;
    __syncthreads();
    float ls = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) ls += wsum[w];
    l = l * al + ls;
    o *= al;
    const int np = (min(tlim - c0, T) + 15) / 16;
#pragma unroll 4
    for (int pg = pw; pg < np; pg += PARTS) {
      const f32x4_any* vr = reinterpret_cast<const f32x4_any*>(
          vp + (static_cast<size_t>(pt[(c0 >> 4) + pg] * a.Hkv + gkv) * HD + d) * 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 v = vr[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float w = sp[pg * 16 + 4 * i + e];
          o = w >= 0.f ? fmaf(w, v[e], o) : o;
        }
      }
    }
    __syncthreads();  // sp and the wave results are rewritten by the next step
  }
  part[pw][d] = o;
  __syncthreads();
  if (pw == 0) {
    float num = o;
#pragma unroll
    for (int i = 1; i < PARTS; ++i) num += part[i][d];
    static_cast<float*>(a.out)[(static_cast<size_t>(r) * a.Hq + h) * HD + d] = num / l;
  }
}

template <int HD, int NT>
void launch_item_kernel(const AttnArgs& a, const AttnItem* items, dim3 grid, int w, hipStream_t st) {
  if (a.tree_base) {
    if (w >= 4) launch_kernel(attn_tree_bf16_kernel<HD, NT, 4>, grid, dim3(4 * kWave), 0, st, a, items);
    else if (w == 2) launch_kernel(attn_tree_bf16_kernel<HD, NT, 2>, grid, dim3(2 * kWave), 0, st, a, items);
    else launch_kernel(attn_tree_bf16_kernel<HD, NT, 1>, grid, dim3(kWave), 0, st, a, items);
    return;
  }
  if (w >= 4) launch_kernel(attn_bf16_kernel<HD, NT, 4>, grid, dim3(4 * kWave), 0, st, a, items);
  else if (w == 2) launch_kernel(attn_bf16_kernel<HD, NT, 2>, grid, dim3(2 * kWave), 0, st, a, items);
  else launch_kernel(attn_bf16_kernel<HD, NT, 1>, grid, dim3(kWave), 0, st, a, items);
}

template <int HD>
hipError_t launch_bf16_hd(const AttnArgs& a, const AttnItem* items, int n_items,
                          const AttnGroup* groups, int n_groups, int nt, int w, hipStream_t st) {
  dim3 grid(n_items * a.Hkv);
  if (n_items > 0) {
    if (nt <= 1) launch_item_kernel<HD, 1>(a, items, grid, w, st);
    else if (nt == 2) launch_item_kernel<HD, 2>(a, items, grid, w, st);
    else launch_item_kernel<HD, 4>(a, items, grid, std::min(w, 2), st);
  }
  if (n_groups > 0) {
    constexpr int DPT = HD == 128 ? 4 : 1;
    attn_combine_kernel<HD, DPT><<<dim3(n_groups, a.Hkv, 16 * nt / kCombineQv), HD / DPT * kCombineQv, 0, st>>>(
        a, groups);
  }
  return hipGetLastError();
}

}  // namespace

const char* attn_kernel_name(int hd, int nt, int w, bool tree) {
  if (tree) {
    static char tnames[2][3][3][48];
    static bool init = false;
    if (!init) {
      for (int h = 0; h < 2; ++h)
        for (int i = 0; i < 3; ++i)
          for (int j = 0; j < 3; ++j)
            snprintf(tnames[h][i][j], sizeof(tnames[h][i][j]), "attn_tree_bf16_kernel<%d, %d, %d>", h ? 128 : 64,
                     1 << i, i == 2 ? std::min(2, 1 << j) : 1 << j);
      init = true;
    }
    return tnames[hd == 128 ? 1 : 0][nt <= 1 ? 0 : (nt == 2 ? 1 : 2)][w <= 1 ? 0 : (w == 2 ? 1 : 2)];
  }
  // [hd 64 / 128][nt 1 / 2 / 4][w 1 / 2 / 4]
  static const char* names[2][3][3] = {
      {{"attn_bf16_kernel<64, 1, 1>", "attn_bf16_kernel<64, 1, 2>", "attn_bf16_kernel<64, 1, 4>"},
       {"attn_bf16_kernel<64, 2, 1>", "attn_bf16_kernel<64, 2, 2>", "attn_bf16_kernel<64, 2, 4>"},
       {"attn_bf16_kernel<64, 4, 1>", "attn_bf16_kernel<64, 4, 2>", "attn_bf16_kernel<64, 4, 2>"}},
      {{"attn_bf16_kernel<128, 1, 1>", "attn_bf16_kernel<128, 1, 2>", "attn_bf16_kernel<128, 1, 4>"},
       {"attn_bf16_kernel<128, 2, 1>", "attn_bf16_kernel<128, 2, 2>", "attn_bf16_kernel<128, 2, 4>"},
       {"attn_bf16_kernel<128, 4, 1>", "attn_bf16_kernel<128, 4, 2>", "attn_bf16_kernel<128, 4, 2>"}}};
  const int i = nt <= 1 ? 0 : (nt == 2 ? 1 : 2);
  const int j = w <= 1 ? 0 : (w == 2 ? 1 : 2);
  return names[hd == 128 ? 1 : 0][i][j];
}

hipError_t launch_attention_bf16(const AttnArgs& a, const AttnItem* d_items, int n_items,
                                 const AttnGroup* d_groups, int n_groups, int nt, int w, hipStream_t st) {
  if (nt > 4 || w > 4) return hipErrorInvalidValue;
  if (a.hd == 128) return launch_bf16_hd<128>(a, d_items, n_items, d_groups, n_groups, nt, w, st);
  if (a.hd == 64) return launch_bf16_hd<64>(a, d_items, n_items, d_groups, n_groups, nt, w, st);
  return hipErrorInvalidValue;
}

hipError_t launch_attention_prefill_bf16(const AttnArgs& a, const AttnItem* d_items, int n_items, bool few_keys,
                                         hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  if (256 % (a.Hq / a.Hkv) || (a.hd != 64 && a.hd != 128)) return hipErrorInvalidValue;
  auto* k = a.hd == 128 ? (few_keys ? attn_prefill_short_bf16_kernel<128> : attn_prefill_bf16_kernel<128>)
                        : (few_keys ? attn_prefill_short_bf16_kernel<64> : attn_prefill_bf16_kernel<64>);
  launch_kernel(k, dim3(n_items * a.Hkv), dim3(512), 0, st, a, d_items);
  return hipGetLastError();
}

const char* attn_prefill_kernel_name(int hd, bool few_keys) {
  if (few_keys) return hd == 128 ? "attn_prefill_short_bf16_kernel<128>" : "attn_prefill_short_bf16_kernel<64>";
  return hd == 128 ? "attn_prefill_bf16_kernel<128>" : "attn_prefill_bf16_kernel<64>";
}

hipError_t launch_attention_f32(const AttnArgs& a, int R, const int32_t* d_row_seq,
                                const int32_t* d_row_pos, hipStream_t st) {
  if (R <= 0) return hipSuccess;
  dim3 grid(R, a.Hq);
  if (a.hd == 64) attn_f32_kernel<64><<<grid, 256, 0, st>>>(a, d_row_seq, d_row_pos);
  else if (a.hd == 128) attn_f32_kernel<128><<<grid, 256, 0, st>>>(a, d_row_seq, d_row_pos);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace spec
