// The layer's flow ratio from the score kernels' sums (FlowMM, Information Flow Guided Merging: rho equation).
#pragma once
#include "device_common.h"
#include "kernels.h"
#include "select_core.h"

namespace flowmm {

// Mean over the query heads of layer l of the share of their proxy attention to sequence b's tokens of the other modality.  One wave
// calls; every workgroup of the layer adds the same numbers in the same order (a kv head's runs, then a tree over the kv heads).
__device__ __forceinline__ float flow_ratio(const Ctx &c, int b, int l) {
  const Shape &sh = c.sh;
  const int *cu = c.meta + c.meta[MW_OFF_CU_SCORE];
  const int x0 = cu[b], x1 = cu[b + 1], lane = threadIdx.x & 63;
  float rho = 0.f;
  for (int h0 = 0; h0 < sh.Hkv; h0 += 64) {
    float v = 0.f;
    if (h0 + lane < sh.Hkv) {
      const float *cp = c.cross_part + (long long)(l * sh.Hkv + h0 + lane) * sh.tiles_score;
      for (int x = x0; x < x1; ++x) v += cp[x];
    }
    rho += wave_sum_dpp(v / (float)sh.W);
  }
  return rho / (float)sh.Hq;
}

}  // namespace flowmm
