// Host-only driver of the projection planner (plan_mfma).  Input lines
// "R N K epi workspace tail" (workspace 0 or 1; tail 0 none, 1 RMSNorm, 2
// rope_kv); output per line "kernel rows w_rows row_tiles w_tiles splits k_len"
// (kernel 2, 3 or 4; rows and W rows of a tile), or "skinny".
#include <cstdio>

#include "gemm_plan.h"

using namespace spec;

int main() {
  int R, N, K, epi, ws, tail;
  while (std::scanf("%d %d %d %d %d %d", &R, &N, &K, &epi, &ws, &tail) == 6) {
    const int Nw = epi == kEpiSwiGLU ? 2 * N : N;
    if (!use_mfma(R, Nw, K)) {
      std::printf("skinny\n");
      continue;
    }
    const size_t bytes = ws ? gemm_splitk_bytes(R, Nw) : 0;
    const MfmaPlan p = plan_mfma(R, N, K, epi, bytes, true, static_cast<Tail>(tail));
    if (p.kernel == MfmaPlan::kM4) {
      const M4Shape& s = kM4Shapes[p.shape];
      std::printf("4 %d %d %d %d %d %d\n", 16 * s.mb, 64 * s.nb, p.tl.MT, p.tl.NT, p.tl.S, p.tl.k_len);
    } else if (p.kernel == MfmaPlan::kM3) {
      const bool small = p.m3.nb != 0;
      std::printf("3 %d %d %d %d %d %d\n", 16 * (small ? kM3sMB : kM3MB), 64 * (small ? p.m3.nb : kM3NB), p.m3.MT,
                  p.m3.NT, p.m3.S, p.m3.k_len);
    } else {
      const int MT = (R + 32 * p.m2.mtw - 1) / (32 * p.m2.mtw), NT = (Nw + 32 * p.m2.ntw - 1) / (32 * p.m2.ntw);
      int k_len = K;
      const int S = mfma2_splits(MT, NT, R, Nw, K, bytes, &k_len);
      std::printf("2 %d %d %d %d %d %d\n", 32 * p.m2.mtw, 32 * p.m2.ntw, MT, NT, S, k_len);
    }
  }
  return 0;
}
