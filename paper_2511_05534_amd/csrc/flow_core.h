// The layer's flow ratio from the score kernels' sums (FlowMM, Information Flow Guided Merging: rho equation).
#pragma once
#include "device_common.h"
#include "kernels.h"

namespace flowmm {

// Mean over the query heads of layer l of the share of their proxy attention to sequence b's tokens of the other modality.  One wave
// calls; every workgroup of the layer adds the same numbers in the same order (a kv head's runs, then the kv heads: read off the lanes that
// hold them, which takes a few cycles each where a walk through LDS waits for every word).
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
    v = v / (float)sh.W;
    const int nh = min(64, sh.Hkv - h0);
    for (int i = 0; i < nh; ++i) rho += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
  }
  return rho / (float)sh.Hq;
}

}  // namespace flowmm
