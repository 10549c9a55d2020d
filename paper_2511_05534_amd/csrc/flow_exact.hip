// The cross-modal interaction ratio with EVERY token of the prompt as a query: the rho^l equation
// of Information Flow Guided Merging taken literally,
//   rho^l = (1/H) sum_h (A_{v->t} + A_{t->v}) / A,   A_{v->t} = sum_{i in V} sum_{j in T} alpha_{i->j}, ...
// with alpha the causal prefill attention of head h (attention equation of the Preliminary
// section) and A the total mass (one per query row).  The proxy-window kernels estimate the same
// ratio from the last W queries only; this one needs the queries of the whole prompt.
//
// Flash-style: the attention matrix is never stored.  A wave holds kFlowRows consecutive query rows of
// one head in registers (MFMA B operand; accumulator rows are keys, so lane n owns query row n of each
// group of 32 and the running softmax statistics of a row are three registers of its lane), and the
// eight waves of a workgroup walk over one stream of keys, which arrives in LDS by direct global->LDS
// loads, double buffered.  The waves of a workgroup take the query heads of the kv group at the same
// positions first, so that they need the same keys; where the grid is small, two or four of them share the
// rows and split the keys, which makes more and shorter workgroups.  Per row: the running maximum, the running sum of
// exp2 and the running sum over IMAGE keys only; the cross-modal mass of the row is the image part for a
// text query and the rest for an image query.  Blocks of 32 keys of one modality (almost all) cost
// nothing extra, and only blocks that reach past the first query row of the wave pay for the causal mask.
//
// What bounds it: a logit costs 16 cycles of matrix core per 64 and about 13 of vector issue
// (v_exp_f32 8, multiply-add 2, add 2, half a maximum), with the clock held down by the power limit.
// Keys in registers and queries in LDS, with the statistics of all 256 rows of the workgroup in every
// wave, held two waves per SIMD; this split needs half the registers and runs four, whose matrix
// and vector phases overlap: 28 layers x 28/4 heads x 4096 tokens 2930 -> 1800 us (935 TFLOP/s; the
// wave's priority raised during its matrix phase is 4 % of that).  Workgroups take groups of units, a group's
// units in turn, the longest key streams first: unit by unit on one XCD each, the last unit's long ones came late (112 units x 28/4
// heads x 2000 tokens 567 -> 470 us; 32 layers x 32/8 heads x 16384 tokens stay at 34 ms).
#include <cfloat>

#include "device_common.h"
#include "kernels.h"
#include "profile.h"
#include "select_core.h"

namespace flowmm {

namespace {

constexpr int kFThreads = kFlowWaves * 64;
// Workgroups of a group of units, to the next eight units (one or more per XCD).  Half of it is one round of the grid: with fewer the
// last long key streams of every group leave compute units idle, with more an XCD's units no longer share its 4 MB L2.  One group per
// eight units | 1024 | 4096 | 16384 | all units in one, bf16, 128 channels, us: 256 units x 4 heads x 16384 tokens 33850 | 33920 | 33770 |
// 35280 | 37210, x 8192 tokens 8990 | 8760 | 8720 | 9310 | 9310; 112 x 7 x 16384 25980 | 25780 | 26040 | 26180 | 26800, x 4096
// 1785 | 1725 | 1712 | 1702 | 1703, x 2000 534 | 482 | 465 | 463 | 463.
constexpr int kFlowGroupWgs = 4096;

struct FlowCall {
  Ctx c;
  FlowExactArgs a;
};

// SPLIT: flow_ksplit waves share the query rows (the loop's bounds cost registers that the kernel for full grids does not have)
template <bool BF16, int D, bool SPLIT>
__global__ __launch_bounds__(kFThreads, 4) void flow_exact_kernel(KernelArgs<FlowCall> k) {
  const Ctx &c = k.a.c;
  const FlowExactArgs &a = k.a.a;
  using CF = Cfg<BF16, D>;
  using TL = KeyTile<BF16, D>;
  constexpr int NCH = CF::NCH, NF = CF::NF;
  constexpr int ROWS = flow_rows(BF16), QS = ROWS / 32;  // query rows of a wave, in groups of 32
  constexpr int KT = TL::kRows;
  constexpr float kLazy = 8.f;  // the running maximum follows once it is 2^8 behind: exact all the same, z stays far below overflow
  extern __shared__ uint4 lds[];  // [2] key tiles

  const Shape &sh = c.sh;
  const ScalarInts meta = first_meta(k, c.meta);
  // Groups of units, a group's units in turn, late positions (long key streams) first.
  const int units = sh.n_layers * sh.Hkv, u0 = blockIdx.x / (a.group * a.wgs_total) * a.group, n_group = min(a.group, units - u0);
  const int rest = blockIdx.x - u0 * a.wgs_total, turn = rest / n_group, unit = u0 + rest - turn * n_group, x = a.wgs_total - 1 - turn;
  const int l = unit / sh.Hkv, gkv = unit - l * sh.Hkv;
  const ScalarInts cu = meta + meta[MW_OFF_CU_FLOWWG];
  const int b = find_seq(cu, meta[MW_BATCH], x);
  const int qb0 = (meta + meta[MW_OFF_CU_FLOWQ])[b];
  const SeqInfo s = load_seq(meta, b);
  const int L = s.L;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  // item i of the sequence: head i % G of the kv group, query rows [ROWS * (i / G), + ROWS)
  const int items = (L + ROWS - 1) / ROWS * sh.G;
  const int ksplit = SPLIT ? sh.flow_ksplit : 1, per_wg = kFlowWaves / ksplit, ks = SPLIT ? wave / per_wg : 0;  // this wave takes every ksplit-th block of 32 keys, from block ks on
  const int first = (x - cu[b]) * per_wg;
  const int mine = first + wave - ks * per_wg, item = min(mine, items - 1);
  const bool active = mine < items;
  const int pb = item / sh.G, h = gkv * sh.G + (item - pb * sh.G);
  const int p0 = pb * ROWS, p_last = active ? min(p0 + ROWS, L) - 1 : -1;
  const int wg_last = min((min(first + per_wg, items) - 1) / sh.G * ROWS + ROWS, L) - 1;  // last position of the workgroup

  // ---- this wave's query rows (clamped past the end of the sequence), through its share of the LDS ----
  uint4 qf[QS][NF];
  const uint4 *Q = reinterpret_cast<const uint4 *>(a.Q) + (long long)l * a.qs_layer + (long long)h * a.qs_head +
                   (long long)(s.tok_off + p0) * a.qs_tok;
  constexpr bool kStagedQ = kFlowWaves * 32 * NCH <= 2 * TL::kChunks;
  if constexpr (kStagedQ) {
#pragma unroll
    for (int g = 0; g < QS; ++g)
      fetch_rows_staged<BF16, D>(Q, (unsigned)a.qs_tok, min(p0 + 32 * g + n, L - 1) - p0, lds + wave * 32 * NCH, qf[g]);
    __syncthreads();  // the key tiles may overwrite the other waves' shares now
  } else {
#pragma unroll
    for (int g = 0; g < QS; ++g) {
      const uint4 *row = Q + (long long)(min(p0 + 32 * g + n, L - 1) - p0) * a.qs_tok + half;
#pragma unroll
      for (int f = 0; f < NF; ++f) qf[g][f] = row[2 * f];
    }
  }

  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)l * sh.ks_layer + (long long)gkv * sh.ks_head +
                   (long long)s.tok_off * sh.ks_tok;
  const float cl = sh.scale_log2e;
  float m[QS], z[QS], zi[QS];  // of query row 32 g + n, over the keys of this half-wave; m starts finite and below every finite logit
#pragma unroll
  for (int g = 0; g < QS; ++g) { m[g] = -FLT_MAX; z[g] = zi[g] = 0.f; }

  const int ntiles = wg_last / KT + 1;
  TL::template request<kFlowWaves>(K, sh.ks_tok, 0, L - 1, lds, wave);
  SpanCursor span(meta, b);
  for (int t = 0; t < ntiles; ++t) {
    __builtin_amdgcn_s_waitcnt(0);  // this wave's part of tile t has landed
    __syncthreads();                // ... and everybody else's; tile t-1 is no longer read
    if (t + 1 < ntiles)
      TL::template request<kFlowWaves>(K, sh.ks_tok, (t + 1) * KT, L - 1, lds + ((t + 1) & 1) * TL::kChunks, wave);
    const char *tile = reinterpret_cast<const char *>(lds + (t & 1) * TL::kChunks);
    const char *rows0 = tile + TL::frag_offset(n, half, 0), *rows1 = tile + TL::frag_offset(n, half, 1);
#pragma unroll 1
    for (int kb = ks; kb < KT / 32; kb += ksplit) {
      const int key0 = t * KT + 32 * kb;
      if (key0 > p_last) break;  // nothing of this wave may see these keys
      f32x16_t acc[QS];
#pragma unroll
      for (int g = 0; g < QS; ++g)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[g][i] = 0.f;
      // one fragment ahead: the other three waves of the SIMD cover the LDS latency, registers are short
      const char *blk0 = rows0 + kb * TL::block_bytes(1), *blk1 = rows1 + kb * TL::block_bytes(1);
      uint4 next = *reinterpret_cast<const uint4 *>(blk0);
      __builtin_amdgcn_s_setprio(1);  // the matrix phase of a wave goes before the vector phases of the three others on its SIMD
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const uint4 kf = next;
        if (f + 1 < NF) next = *reinterpret_cast<const uint4 *>((f & 1 ? blk0 : blk1) + 64 * ((f + 1) >> 1));
#pragma unroll
        for (int g = 0; g < QS; ++g) mma_chunk<BF16>(acc[g], kf, qf[g][f]);  // [key][query row]
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
      const bool masked = key0 + 31 > p0;
      const unsigned img = span.mask(key0, L);
#pragma unroll
      for (int g = 0; g < QS; ++g) {
        if (masked) {
          const int ln = lane_id_here();
          const int limit = p0 + 32 * g + (ln & 31) - key0 - 4 * (ln >> 5);  // row i of the block may be seen up to here
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[g][i] = acc_row(i, 0) <= limit ? acc[g][i] : -INFINITY;
        }
        float tm = fmaxf(acc[g][0], acc[g][1]);
#pragma unroll
        for (int i = 2; i < 16; i += 2) tm = fmaxf(fmaxf(tm, acc[g][i]), acc[g][i + 1]);
        tm *= cl;  // cl > 0: the largest logit is the largest product
        if (__any(tm > m[g] + kLazy)) {
          const float M = fmaxf(m[g], tm), sc = fast_exp2(m[g] - M);
          z[g] *= sc;
          zi[g] *= sc;
          m[g] = M;
        }
        float za = 0.f, zb = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          acc[g][i] = fast_exp2(fmaf(acc[g][i], cl, -m[g]));
          acc[g][i + 1] = fast_exp2(fmaf(acc[g][i + 1], cl, -m[g]));
          za += acc[g][i];
          zb += acc[g][i + 1];
        }
        za += zb;
        if (img == 0xffffffffu) {
          zi[g] += za;
        } else if (img != 0u) {  // both modalities in this block (rare)
          const unsigned mine = img >> (4 * half);
#pragma unroll
          for (int i = 0; i < 16; ++i) zi[g] += (mine >> acc_row(i, 0)) & 1u ? acc[g][i] : 0.f;
        }
        z[g] += za;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- fold the two half-waves, then the waves with the same rows; the share of every row; their sum (a fixed tree) ----
  auto fold = [&](int g, float m2, float z2, float zi2) {
    const float M = fmaxf(m[g], m2), s1 = fast_exp2(m[g] - M), s2 = fast_exp2(m2 - M);
    z[g] = z[g] * s1 + z2 * s2;
    zi[g] = zi[g] * s1 + zi2 * s2;
    m[g] = M;
  };
#pragma unroll
  for (int g = 0; g < QS; ++g) fold(g, __shfl_xor(m[g], 32, 64), __shfl_xor(z[g], 32, 64), __shfl_xor(zi[g], 32, 64));
  if constexpr (SPLIT) {
    __syncthreads();  // nobody reads keys any more
    float4 *lds_stat = reinterpret_cast<float4 *>(lds);  // [waves][ROWS]
#pragma unroll
    for (int g = 0; g < QS; ++g)
      if (half == 0) lds_stat[wave * ROWS + 32 * g + n] = make_float4(m[g], z[g], zi[g], 0.f);
    __syncthreads();
    if (ks > 0) return;
#pragma unroll
    for (int g = 0; g < QS; ++g)
      for (int w = wave + per_wg; w < kFlowWaves; w += per_wg) {
        const float4 o = lds_stat[w * ROWS + 32 * g + n];
        fold(g, o.x, o.y, o.z);
      }
  }
  if (!active) return;
  float share = 0.f;
  SpanCursor rows(meta, b);
#pragma unroll
  for (int g = 0; g < QS; ++g) {
    const int q = p0 + 32 * g + n;
    const unsigned img = p0 + 32 * g < L ? rows.mask(p0 + 32 * g, L) : 0u;
    if (half == 0 && q < L && z[g] > 0.f) share += ((img >> n) & 1u ? z[g] - zi[g] : zi[g]) / z[g];  // mass sent to the other modality
  }
  share = wave_sum(share);
  if (lane == 0) a.part[((long long)l * sh.Hq + h) * a.qblocks_total + qb0 + pb] = share;
}

// rho of every (layer, sequence): a wave adds the query blocks of its heads, lane j taking blocks j, j + 64, ..; then the waves in order
__global__ __launch_bounds__(1024) void flow_exact_finish_kernel(KernelArgs<FlowCall> k) {
  const Ctx &c = k.a.c;
  const FlowExactArgs &a = k.a.a;
  __shared__ float lds_wave[16];
  const Shape &sh = c.sh;
  const ScalarInts meta = first_meta(k, c.meta);
  const int b = blockIdx.x, l = blockIdx.y;
  const ScalarInts cu = meta + meta[MW_OFF_CU_FLOWQ];
  const int x0 = cu[b], x1 = cu[b + 1];
  const SeqInfo s = load_seq(meta, b);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float acc = 0.f;
  for (int h = wave; h < sh.Hq; h += 16) {
    const float *part = a.part + ((long long)l * sh.Hq + h) * a.qblocks_total;
    float v = 0.f;
    for (int x = x0 + lane; x < x1; x += 64) v += part[x];
    acc += wave_sum(v) / (float)s.L;
  }
  if (lane == 0) lds_wave[wave] = acc;
  __syncthreads();
  if (threadIdx.x != 0) return;
  float rho = 0.f;
  for (int w = 0; w < 16; ++w) rho += lds_wave[w];
  rho /= (float)sh.Hq;
  a.rho[l * sh.batch + b] = rho;
  a.mode[l * sh.batch + b] = (rho > sh.theta) != (sh.invert_flow != 0) ? 1 : 0;
}

template <bool BF16, int D>
hipError_t launch_flow_exact_t(const Ctx &c, FlowExactArgs a, const int *words, int n_words) {
  static_assert(kFlowWaves * flow_rows(BF16) <= 2 * KeyTile<BF16, D>::kChunks, "the waves' statistics take the place of the keys");
  const size_t lds = 2 * (size_t)KeyTile<BF16, D>::kChunks * 16;
  const bool split = c.sh.flow_ksplit > 1;
  hipError_t e = split ? allow_full_lds<flow_exact_kernel<BF16, D, true>>() : allow_full_lds<flow_exact_kernel<BF16, D, false>>();
  if (e != hipSuccess) return e;
  const int units = c.sh.n_layers * c.sh.Hkv;
  const long long grid = (long long)units * a.wgs_total;
  if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  a.group = (kFlowGroupWgs / a.wgs_total + 7) / 8 * 8;
  if (a.group < 8) a.group = 8;
  if (a.group > units) a.group = units;
  KernelArgs<FlowCall> k;
  fill_kernel_args(k, FlowCall{c, a}, words, n_words);
  {
    ProfScope ps(c.stream, KID_FLOW_EXACT);
    if (split) flow_exact_kernel<BF16, D, true><<<dim3((unsigned)grid), kFThreads, lds, c.stream>>>(k);
    else flow_exact_kernel<BF16, D, false><<<dim3((unsigned)grid), kFThreads, lds, c.stream>>>(k);
  }
  flow_exact_finish_kernel<<<dim3(c.sh.batch, c.sh.n_layers), 1024, 0, c.stream>>>(k);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_flow_exact(const Ctx &c, const FlowExactArgs &a, const int *words, int n_words) {
  if (c.sh.bf16) return c.sh.d == 128 ? launch_flow_exact_t<true, 128>(c, a, words, n_words) : launch_flow_exact_t<true, 64>(c, a, words, n_words);
  return c.sh.d == 128 ? launch_flow_exact_t<false, 128>(c, a, words, n_words) : launch_flow_exact_t<false, 64>(c, a, words, n_words);
}

}  // namespace flowmm
