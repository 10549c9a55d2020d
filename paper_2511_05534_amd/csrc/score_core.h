// Pieces of the score kernels that contract query rows staged in LDS with keys held in registers (score.hip).
#pragma once
#include "device_common.h"

namespace flowmm {

// The products of one block of 32 query rows with this wave's keys (bf16).  KEYS_AS_ROWS: accumulator
// rows are keys and lane n owns query row n (pass 1); otherwise rows are query rows and lane n owns
// key n of every group (pass 3).  Fragments are requested kAhead steps ahead, also across blocks.
template <int D, int KS, bool KEYS_AS_ROWS, int AHEAD>
__device__ __forceinline__ void block_products(f32x16_t (&acc)[KS], const RowOperand<Cfg<true, D>::NF, kPlain> (&kf)[KS],
                                               uint4 (&pf)[AHEAD], const char *qrow, bool more) {
  constexpr int NF = Cfg<true, D>::NF, RS = Cfg<true, D>::NCH + 1;
#pragma unroll
  for (int sub = 0; sub < KS; ++sub)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[sub][i] = 0.f;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const uint4 cur = pf[f % AHEAD];
    if (f + AHEAD < NF) pf[f % AHEAD] = *reinterpret_cast<const uint4 *>(qrow + 32 * (f + AHEAD));
#pragma unroll
    for (int sub = 0; sub < KS; ++sub) {
      if constexpr (KEYS_AS_ROWS) mma_chunk<true>(acc[sub], kf[sub].f[f], cur);
      else mma_chunk<true>(acc[sub], cur, kf[sub].f[f]);
    }
  }
  if (more) {
#pragma unroll
    for (int f = 0; f < AHEAD; ++f) pf[f] = *reinterpret_cast<const uint4 *>(qrow + 32 * RS * 16 + 32 * f);
  }
}

}  // namespace flowmm
