// Unit-resident path for short prompts (every L <= 1024, or 384 to 1024 in fp32: unit_max_tokens; G*W <= 64, every B <= 256,
// at most 8 sequences and 32 modality spans, whose description rides in the kernel arguments).
//
// When one (sequence, layer, kv head) unit fits on a compute unit, every step of a unit runs inside
// one workgroup and nothing but K, V and the results touches HBM:
//   unit_plan   : proxy attention -> importance, top-B split, cosine argmax as a cross-modal layer
//                 does; the unit's keys stay in registers throughout (K read once)
//   unit_match  : the layer's flow ratio and strategy (needs all its query heads, hence its own
//                 launch); units of intra-modal layers are split and matched again with the
//                 modality restriction, the others return at once
//   unit_merge  : counting sort + segment sums    (K and V read once)
// The generic path's plans of up to 2048 tokens are merged by unit_merge too where there are units enough (unit_merge_fits).
// Three launches, two in the one-call entry point, where the generic kernels take three to six (one fp32 layer of 4 heads x 320 tokens, one call and
// two: 36.6 and 39.3 us through the generic kernels, 29.2 and 31.1 here).  The arithmetic is the same as in the generic kernels
// (score.hip, select.hip, match.hip, merge.hip); see those files for the paper passages.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "profile.h"
#include "select_core.h"
#include "unit_merge_core.h"

namespace flowmm {

namespace {

// ============================ score + select + match (cross-modal) ===========================
// One workgroup of WAVES (eight or twelve) waves per unit; PAIR: two such workgroups per compute unit.  Wave w keeps the key tiles w, w+WAVES, ... (32 keys each) in
// registers for the whole kernel, in the layout every contraction here uses, so K is read from
// HBM once.  The logits are computed twice from those registers: once for the row statistics,
// once for the normalised column sums.  The pivots' rows go from the registers of the lanes that
// hold them to LDS, and the same registers are the token operands of the cosine contraction.
// Every fragment read from LDS (query rows, pivot rows) feeds one matrix instruction per tile of
// the wave.  The layer's strategy needs all its query heads and is not known here: this kernel
// matches as a cross-modal layer does; unit_match_kernel then settles the strategy and redoes the
// intra-modal layers.
constexpr int kPMaxWaves = 12;  // workgroups of 8 or 12 waves (12 * 154 registers still fit a compute unit)

struct PlanLds {  // byte offsets into the dynamic LDS block
  int q, stat, cval, rowimg, limit, cross, keys, assign, kept, piv, w, bias, total_bytes;
};

__host__ __device__ inline PlanLds plan_lds_layout(int rows, int b_pad, int nch) {
  PlanLds m;
  int off = 0;
  m.q = off; off += rows * (nch + 1) * 16;
  m.piv = off; off += b_pad * (nch + 1) * 16;
  m.stat = off; off += kPMaxWaves * rows * 8;
  m.cval = off; off += rows * 4;
  m.rowimg = off; off += rows * 4;
  m.limit = off; off += rows * 4;
  m.cross = off; off += 32 * 2 * 4;
  m.keys = off; off += 1024 * 4;
  m.assign = off; off += 1024 * 4;
  m.kept = off; off += b_pad * 4;
  m.w = off; off += b_pad * 4;
  m.bias = off; off += b_pad * 4;
  m.total_bytes = (off + 15) & ~15;
  return m;
}

// Waves per SIMD that the registers are shared among.  One key tile a wave: six, two workgroups of twelve waves or three of eight on a compute unit (bf16, with
// the 84 registers that the compiler takes by itself one and two: calls with 1024 units x 300 tokens 75.6 -> 88.5 us); fp32 rows of 128 channels four, two
// workgroups of eight waves; as many as there are of fp32 rows split into terms.
template <bool BF16, int D, int NT, bool PAIR, Operand KEYS>
constexpr int plan_waves_per_simd() { return PAIR ? 4 : NT > 1 || KEYS != kPlain ? 1 : BF16 || D == 64 ? 6 : 4; }

template <bool BF16, int D, int RB, int NT, int WAVES, bool PAIR, Operand KEYS>
__global__ __launch_bounds__(WAVES * 64, (plan_waves_per_simd<BF16, D, NT, PAIR, KEYS>())) void unit_plan_kernel(Ctx c, int b_pad) {
  constexpr int NJ = PAIR ? 1 : NT;  // key tiles in the accumulators at a time
  constexpr int NR = PAIR && NT > 2 ? 2 : NT;  // key tiles of a wave that stay in registers; the third comes out of the L2 in every pass
  constexpr int kPThreads = WAVES * 64, kPWaves = WAVES;
  using CF = Cfg<BF16, D>;
  constexpr int NCH = CF::NCH, NF = CF::NF, RS = NCH + 1;
  constexpr int ROWS = RB * 32;
  extern __shared__ __align__(16) char lds_dyn[];
  const PlanLds lay = plan_lds_layout(ROWS, b_pad, NCH);
  uint4 *ldsq = reinterpret_cast<uint4 *>(lds_dyn + lay.q);            // [ROWS][RS] query rows
  uint4 *lds_piv = reinterpret_cast<uint4 *>(lds_dyn + lay.piv);       // [b_pad][RS] pivot rows
  float2 *lds_stat = reinterpret_cast<float2 *>(lds_dyn + lay.stat);   // [waves][ROWS] (max, sum exp2)
  float *lds_c = reinterpret_cast<float *>(lds_dyn + lay.cval);        // [ROWS] max + log2(sum)
  float *lds_rowimg = reinterpret_cast<float *>(lds_dyn + lay.rowimg); // [ROWS] 1 for an image proxy row
  int *lds_limit = reinterpret_cast<int *>(lds_dyn + lay.limit);       // [ROWS] last key a proxy row may see, -1 for a padding row
  float *lds_cross = reinterpret_cast<float *>(lds_dyn + lay.cross);   // [tiles][RB] cross-modal mass per key tile
  unsigned *lds_keys = reinterpret_cast<unsigned *>(lds_dyn + lay.keys);  // [1024] importance bits
  int *lds_assign = reinterpret_cast<int *>(lds_dyn + lay.assign);     // [1024] slot of a pivot, -2 otherwise
  int *lds_kept = reinterpret_cast<int *>(lds_dyn + lay.kept);         // [B]
  float *lds_w = reinterpret_cast<float *>(lds_dyn + lay.w);           // [b_pad] 1/norm (0 for a zero row)
  float *lds_bias = reinterpret_cast<float *>(lds_dyn + lay.bias);     // [b_pad] added to a candidate
  __shared__ SmallSelectScratch<kPThreads> scratch;
  __shared__ int sh_dropped;

  const Shape &sh = c.sh;
  const int b = rotated_block_x(), gkv = blockIdx.y, l = blockIdx.z + c.layer0;
  const SeqInfo s = inline_seq(c.inl, b);
  const int L = s.L;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  const long long unit = (long long)l * sh.Hkv + gkv;

  // ---- every key of the unit into registers ----------------------------------------------------
  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)l * sh.ks_layer +
                   (long long)gkv * sh.ks_head + (long long)s.tok_off * sh.ks_tok;
  uint4 kf[NR][NF];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int key0 = (wave + kPWaves * j) * 32;
    if (key0 < L) {
      const uint4 *row = K + (long long)min(key0 + n, L - 1) * sh.ks_tok + half;
#pragma unroll
      for (int f = 0; f < NF; ++f) kf[j][f] = row[2 * f];
    } else {
#pragma unroll
      for (int f = 0; f < NF; ++f) kf[j][f] = make_uint4(0, 0, 0, 0);
    }
  }
  // the query rows, the heads' windows next to each other (zero rows pad them to whole blocks of 32)
  const int R = sh.G * sh.W;
  {
    const uint4 *Q = reinterpret_cast<const uint4 *>(c.Q) + (long long)l * sh.qs_layer;
    for (int idx = threadIdx.x; idx < ROWS * NCH; idx += kPThreads) {
      const int row = idx / NCH, ch = idx - row * NCH;
      const int g = row / sh.W, r = row - g * sh.W;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (row < R) v = Q[(long long)(gkv * sh.G + g) * sh.qs_head + (long long)(b * sh.W + r) * sh.qs_tok + ch];
      ldsq[row * RS + ch] = v;
    }
    for (int row = threadIdx.x; row < ROWS; row += kPThreads) {
      const int r = window_row(sh, row);
      lds_rowimg[row] = (row < R && inline_mod(c.inl, b, L - sh.W + r)) ? 1.f : 0.f;
      lds_limit[row] = row < R ? L - sh.W + r : -1;
    }
    if (threadIdx.x == 0) sh_dropped = 0;
  }
  __syncthreads();

  constexpr bool kSplit = KEYS == kSplitOnce;
  static_assert(!kSplit || (!BF16 && NT == 1), "registers for one split key tile a wave");
  RowOperand<NF, KEYS> keys[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) keys[j].set(kf[j]);
  auto key_row = [&](int j) { return K + (long long)min((wave + kPWaves * j) * 32 + (lane_id_here() & 31), L - 1) * sh.ks_tok + (lane_id_here() >> 5); };
  // products of NJ key tiles from j0 on with 32 rows in LDS (this lane's first fragment at rows); keys_first: the tile's rows are keys
  auto tile_products = [&](f32x16_t (&acc)[NJ], int j0, const uint4 *rows, auto keys_first) {
    constexpr bool kFirst = decltype(keys_first)::value;
    auto mma = [](f32x16_t &d, const uint4 &k, const uint4 &o) {
      if constexpr (kFirst) mma_chunk<BF16>(d, k, o);
      else mma_chunk<BF16>(d, o, k);
    };
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[jj][i] = 0.f;
    if (PAIR && (wave + kPWaves * j0) * 32 >= L) return;  // no such tile
    if constexpr (!BF16) {
      auto other = [&](int f) { return rows[2 * f]; };
      if (j0 >= NR) {
        RowOperand<NF, kPlain> far[1];
        const uint4 *row = key_row(j0);
#pragma unroll
        for (int f = 0; f < NF; ++f) far[0].f[f] = row[2 * f];
        f32x16_t one[1];
        f32_products<kFirst>(one, far, other, [&](int, int f) { return row[2 * f]; });
        acc[0] = one[0];
      } else {
        f32_products<kFirst>(acc, keys + j0, other, [&](int jj, int f) { return key_row(j0 + jj)[2 * f]; });
      }
      return;
    }
    if (j0 >= NR) {
      const uint4 *row = key_row(j0);
      constexpr int NW = 4;  // fragments in flight
#pragma unroll
      for (int f0 = 0; f0 < NF; f0 += NW) {
        uint4 kw[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) kw[i] = row[2 * (f0 + i)];
#pragma unroll
        for (int i = 0; i < NW; ++i) mma(acc[0], kw[i], rows[2 * (f0 + i)]);
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const uint4 q = rows[2 * f];
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) mma(acc[jj], kf[j0 + jj][f], q);
      if (PAIR && f % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // two fragments at a time, not all of them: registers are short
    }
  };
  const float cl = sh.scale_log2e;
  const uint4 *qlane = ldsq + n * RS + half;  // this lane's first fragment of row block 0
  // ---- pass 1: row statistics; accumulator rows are keys, lane n owns query row rb*32+n ----------
  // Only the tiles that reach into the window (or past the end) pay for the causal mask.
  {
    float m[RB], z[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) { m[rb] = -INFINITY; z[rb] = 0.f; }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int limit = lds_limit[rb * 32 + n];  // last key this query may see
#pragma unroll
      for (int j0 = 0; j0 < NT; j0 += NJ) {
        f32x16_t acc[NJ];
        tile_products(acc, j0, qlane + rb * 32 * RS, std::true_type{});  // [key][query row]
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
          const int key0 = (wave + kPWaves * (j0 + jj)) * 32;
          if (key0 >= L) continue;
          float tm = -INFINITY;
          if (key0 + 31 > L - sh.W) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              acc[jj][i] = key0 + acc_row(i, half) <= limit ? acc[jj][i] : -INFINITY;
              tm = fmaxf(tm, acc[jj][i]);
            }
          } else {
#pragma unroll
            for (int i = 0; i < 16; i += 2) tm = fmaxf(fmaxf(tm, acc[jj][i]), acc[jj][i + 1]);
          }
          if (tm > -INFINITY) {
            const float M = fmaxf(m[rb], tm * cl);  // cl > 0: the largest logit is the largest product
            float zt = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) zt += fast_exp2(fmaf(acc[jj][i], cl, -M));
            z[rb] = z[rb] * fast_exp2(m[rb] - M) + zt;
            m[rb] = M;
          }
          if constexpr (PAIR) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float m2 = __shfl_xor(m[rb], 32, 64), z2 = __shfl_xor(z[rb], 32, 64);
      stat_combine(m[rb], z[rb], m2, z2);
      if (half == 0) lds_stat[wave * ROWS + rb * 32 + n] = make_float2(m[rb], z[rb]);
    }
  }
  __syncthreads();
  if (threadIdx.x < ROWS) {
    float2 a = lds_stat[threadIdx.x];
#pragma unroll
    for (int w = 1; w < kPWaves; ++w) {
      const float2 o = lds_stat[w * ROWS + threadIdx.x];
      stat_combine(a.x, a.y, o.x, o.y);
    }
    // exp2(logit - c) is the normalised probability; padding rows get c = +inf, probability 0
    lds_c[threadIdx.x] = (int)threadIdx.x < R && a.y > 0.f ? a.x + __builtin_amdgcn_logf(a.y) : INFINITY;
  }
  __syncthreads();

  // ---- pass 2: probabilities reduced over the query rows; rows are query rows, lane n owns key n --
  {
    const float inv_rows = 1.0f / (float)(sh.G * sh.W);
    float *imp = c.importance + unit * sh.T + s.tok_off;
    const bool win_img = s.win_has_img != 0;
#pragma unroll
    for (int j0 = 0; j0 < NT; j0 += NJ) {
      float colsum[NJ];
      int keymod[NJ];
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) {
        colsum[jj] = 0.f;
        keymod[jj] = inline_mod(c.inl, b, min((wave + kPWaves * (j0 + jj)) * 32 + n, L - 1));
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        f32x16_t acc[NJ];
        tile_products(acc, j0, qlane + rb * 32 * RS, std::false_type{});  // [query row][key]
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
          const int key0 = (wave + kPWaves * (j0 + jj)) * 32;
          if (key0 >= L) continue;
          const int key = key0 + n;
          float bs = 0.f, bsi = 0.f;
          const bool general = win_img || key0 + 31 > L - sh.W;  // causal mask, image rows in the window
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const float4 c4 = *reinterpret_cast<const float4 *>(lds_c + rb * 32 + 8 * g + 4 * half);
            const float cr[4] = {c4.x, c4.y, c4.z, c4.w};
            if (general) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int row = rb * 32 + 8 * g + 4 * half + i;
                float p = fast_exp2(fmaf(acc[jj][4 * g + i], cl, -cr[i]));  // padding rows: c = +inf, p = 0
                p = key <= lds_limit[row] ? p : 0.f;
                bs += p;
                bsi = fmaf(p, lds_rowimg[row], bsi);
              }
            } else {
#pragma unroll
              for (int i = 0; i < 4; ++i) bs += fast_exp2(fmaf(acc[jj][4 * g + i], cl, -cr[i]));
            }
            if constexpr (PAIR) __builtin_amdgcn_sched_barrier(0);
          }
          colsum[jj] += bs;
          // mass on keys of the other modality: image keys seen by text rows, text keys by image rows
          const float cross = wave_sum(keymod[jj] ? bs - bsi : bsi);
          if (lane == 0) lds_cross[(key0 >> 5) * RB + rb] = cross;
        }
      }
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) {
        const int key = (wave + kPWaves * (j0 + jj)) * 32 + n;
        const float tot = (colsum[jj] + __shfl_xor(colsum[jj], 32, 64)) * inv_rows;
        if (half == 0 && key < L) {
          imp[key] = tot;
          lds_keys[key] = __float_as_uint(tot);
        }
      }
      if constexpr (PAIR) __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();
  if (wave == 0) {
    // lane t adds tile t's share, then a fixed tree over the lanes (the same for every shape of workgroup)
    float v = 0.f;
    if (lane < ((L + 31) >> 5))
      for (int rb = 0; rb < RB; ++rb) v += lds_cross[lane * RB + rb];
    v = wave_sum(v);
    if (lane == 0) c.cross_part[unit * sh.tiles_score + b] = v;
  }

  // ---- top-B split ---------------------------------------------------------------------------------
  {
    unsigned keys4[4];  // every thread's four consecutive keys (threads past the end hold none)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = threadIdx.x * 4 + j;
      keys4[j] = i < L ? lds_keys[i] : 0u;
    }
    select_top_b_small<kPThreads>(keys4, L, sh.W, s.B, lds_kept, lds_assign, scratch);
    for (int idx = s.B * NCH + (int)threadIdx.x; idx < b_pad * NCH; idx += kPThreads)  // padding pivot rows
      lds_piv[(idx / NCH) * RS + idx % NCH] = make_uint4(0, 0, 0, 0);
  }
  __syncthreads();
  int *kept = c.kept_idx + unit * sh.SB + s.kept_off;
  for (int i = threadIdx.x; i < s.B; i += kPThreads) kept[i] = lds_kept[i];

  // ---- pivots: rows from the registers that hold them, then inverse norms and the sensitivity gate ----
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int tok = (wave + kPWaves * j) * 32 + n;
    const int slot = tok < L ? lds_assign[tok] : -2;
    if (slot >= 0) {
      if (j < NR && !kSplit) {
#pragma unroll
        for (int f = 0; f < NF; ++f) lds_piv[slot * RS + 2 * f + half] = kf[j < NR ? j : 0][f];
      } else {
        const uint4 *row = K + (long long)tok * sh.ks_tok + half;
#pragma unroll
        for (int f = 0; f < NF; ++f) lds_piv[slot * RS + 2 * f + half] = row[2 * f];
      }
    }
  }
  __syncthreads();
  for (int pr0 = 0; pr0 < b_pad; pr0 += kPThreads / NCH) {  // NCH lanes per row
    const int pr = pr0 + threadIdx.x / NCH, ch = threadIdx.x % NCH;
    float ss = pr < b_pad ? chunk_sumsq<BF16>(lds_piv[pr * RS + ch]) : 0.f;
#pragma unroll
    for (int o = NCH / 2; o >= 1; o >>= 1) ss += __shfl_xor(ss, o, 64);
    if (ch == 0 && pr < b_pad) {
      const bool ok = pr < s.B && !(__uint_as_float(lds_keys[lds_kept[pr < s.B ? pr : 0]]) > s.tau);
      lds_w[pr] = inverse_norm(ss);
      // added to every candidate: keeps an eligible one a normal float, sinks the others
      lds_bias[pr] = ok ? 1e-30f : -3e38f;
    }
  }
  __syncthreads();

  // ---- match as a cross-modal layer does ---------------------------------------------------------------
  // Each candidate is cosine * |token| (+ bias); its low four mantissa bits are replaced by 15 - i,
  // i the row inside this lane's 16 rows of the block, so one running maximum carries the argmax.
  int *assign = c.assign + unit * sh.T + s.tok_off;
  const int nblk = b_pad >> 5;
  int dropped = 0;
  const uint4 *plane = lds_piv + n * RS + half;
#pragma unroll
  for (int j0 = 0; j0 < NT; j0 += NJ) {
    float best[NJ];
    int best_blk[NJ];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) { best[jj] = -INFINITY; best_blk[jj] = 0; }
    for (int pb = 0; pb < nblk; ++pb) {
      f32x16_t acc[NJ];
      tile_products(acc, j0, plane + pb * 32 * RS, std::false_type{});  // [pivot][token]
      float m[NJ];
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) m[jj] = -INFINITY;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 w4 = *reinterpret_cast<const float4 *>(lds_w + pb * 32 + 8 * g + 4 * half);
        const float4 b4 = *reinterpret_cast<const float4 *>(lds_bias + pb * 32 + 8 * g + 4 * half);
        const float wv[4] = {w4.x, w4.y, w4.z, w4.w}, bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
          for (int k = 0; k < 4; k += 2) {
            const int i = 4 * g + k;
            const float p0 = __uint_as_float((__float_as_uint(fmaf(acc[jj][i], wv[k], bv[k])) & ~15u) | (unsigned)(15 - i));
            const float p1 = __uint_as_float((__float_as_uint(fmaf(acc[jj][i + 1], wv[k + 1], bv[k + 1])) & ~15u) | (unsigned)(14 - i));
            m[jj] = fmaxf(fmaxf(m[jj], p0), p1);
          }
        if constexpr (PAIR) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj)
        if (m[jj] > best[jj]) { best[jj] = m[jj]; best_blk[jj] = pb; }
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const int tok = (wave + kPWaves * (j0 + jj)) * 32 + n;
      int best_slot = best_blk[jj] * 32 + acc_row(15 - (int)(__float_as_uint(best[jj]) & 15u), half);
      const float ob = __shfl_xor(best[jj], 32, 64);
      const int os = __shfl_xor(best_slot, 32, 64);
      float bj = best[jj];
      if (ob > bj || (ob == bj && os < best_slot)) { bj = ob; best_slot = os; }
      if (!(bj > -1e38f)) best_slot = -1;  // no eligible pivot
      if (half == 0 && tok < L) {
        const int cur = lds_assign[tok];
        assign[tok] = cur == -2 ? best_slot : cur;  // a pivot keeps its own slot
        dropped += cur == -2 && best_slot < 0;
      }
    }
    if constexpr (PAIR) __builtin_amdgcn_sched_barrier(0);
  }
  dropped = wave_sum_int(dropped);
  if (lane == 0 && dropped) atomicAdd(&sh_dropped, dropped);
  __syncthreads();
  if (threadIdx.x == 0) c.n_dropped[unit * sh.batch + b] = sh_dropped;
}

// ============================ flow (+ select + match of intra-modal layers) ====================
struct MatchLds {  // byte offsets into the dynamic LDS block
  int piv, w, bias, keys, assign, kept, total_bytes;
};

__host__ __device__ inline MatchLds match_lds_layout(int b_pad, int nch, int maxL) {
  MatchLds m;
  int off = 0;
  m.piv = off; off += b_pad * (nch + 1) * 16;
  m.w = off; off += b_pad * 4;
  m.bias = off; off += 2 * b_pad * 4;
  m.keys = off; off += maxL * 4;
  m.assign = off; off += maxL * 4;
  m.kept = off; off += b_pad * 4;
  m.total_bytes = (off + 15) & ~15;
  return m;
}

// Whether layer l merges across modalities in sequence b.  Every wave of the layer's workgroups adds the kv heads' shares in the same tree; nothing waits
// for another wave.  (One after the other, read off the lanes that hold them: 0.6 us more with 32 heads.)
__device__ __forceinline__ bool unit_flow(const Ctx &c, int b, int gkv, int l) {
  const Shape &sh = c.sh;
  const int lane = threadIdx.x & 63;
  float acc = 0.f;
  for (int h0 = 0; h0 < sh.Hkv; h0 += 64) {
    const float v = h0 + lane < sh.Hkv ? c.cross_part[(long long)(l * sh.Hkv + h0 + lane) * sh.tiles_score + b] / (float)sh.W : 0.f;
    acc += wave_sum_dpp(v);
  }
  const float rho = acc / (float)sh.Hq;
  const bool cross = (rho > sh.theta) != (sh.invert_flow != 0);
  if (gkv == 0 && threadIdx.x == 0) {
    c.rho[l * sh.batch + b] = rho;
    c.mode[l * sh.batch + b] = cross ? 1 : 0;
  }
  return cross;
}

// An intra-modal layer's unit (b, gkv, l): the split again (same result) and the match restricted to the token's modality.  All threads of the
// workgroup call; lds_dyn: match_lds_layout bytes.
template <bool BF16, int D, int THREADS>
__device__ __forceinline__ void unit_intra_match_body(const Ctx &c, int b_pad, char *lds_dyn, int b, int gkv, int l) {
  constexpr int kF2Threads = THREADS, kF2Waves = THREADS / 64;
  using CF = Cfg<BF16, D>;
  constexpr int NCH = CF::NCH, NF = CF::NF;
  const MatchLds lay = match_lds_layout(b_pad, NCH, c.sh.maxL);
  uint4 *lds_piv = reinterpret_cast<uint4 *>(lds_dyn + lay.piv);     // [b_pad][NCH+1] pivot rows
  float *lds_w = reinterpret_cast<float *>(lds_dyn + lay.w);         // [b_pad] 1/norm (0 for a zero row)
  float *lds_bias = reinterpret_cast<float *>(lds_dyn + lay.bias);   // [2][b_pad] 0 eligible, -inf not
  unsigned *lds_keys = reinterpret_cast<unsigned *>(lds_dyn + lay.keys);  // [L] importance bits
  int *lds_assign = reinterpret_cast<int *>(lds_dyn + lay.assign);   // [L] slot of a pivot, -2 otherwise
  int *lds_kept = reinterpret_cast<int *>(lds_dyn + lay.kept);       // [B]
  __shared__ SmallSelectScratch<kF2Threads> scratch;
  __shared__ int sh_dropped;

  const Shape &sh = c.sh;
  const SeqInfo s = inline_seq(c.inl, b);
  const int L = s.L;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  const long long unit = (long long)l * sh.Hkv + gkv;
  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)l * sh.ks_layer +
                   (long long)gkv * sh.ks_head + (long long)s.tok_off * sh.ks_tok;
  const unsigned *imp = reinterpret_cast<const unsigned *>(c.importance) + unit * sh.T + s.tok_off;
  int *kept = c.kept_idx + unit * sh.SB + s.kept_off;
  int *assign = c.assign + unit * sh.T + s.tok_off;

  if (threadIdx.x == 0) sh_dropped = 0;  // (the split below has barriers)

  const int ntiles = (L + 31) >> 5;
  uint4 kf[NF];
  int t = wave;
  if (t < ntiles) {
    const uint4 *row = K + (long long)min(t * 32 + n, L - 1) * sh.ks_tok + half;
#pragma unroll
    for (int f = 0; f < NF; ++f) kf[f] = row[2 * f];
  }
  unsigned keys4[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = threadIdx.x * 4 + j;
    keys4[j] = i < L ? imp[i] : 0u;
    if (i < L) lds_keys[i] = keys4[j];
  }
  // top-B split (pivot list and pivot/non-pivot marks stay in LDS; the plan gets its copy below)
  select_top_b_small<kF2Threads>(keys4, L, sh.W, s.B, lds_kept, lds_assign, scratch);
  __syncthreads();
  for (int i = threadIdx.x; i < s.B; i += kF2Threads) kept[i] = lds_kept[i];

  // stage all pivots once: rows, inverse norms, eligibility per token modality
  constexpr int kRowsPerPass = kF2Threads / NCH;
  for (int r0 = 0; r0 < b_pad; r0 += kRowsPerPass) {
    const int pr = r0 + threadIdx.x / NCH, ch = threadIdx.x % NCH;
    uint4 v = make_uint4(0, 0, 0, 0);
    const bool real = pr < s.B;
    const int ptok = real ? lds_kept[pr] : 0;
    if (real) v = K[(long long)ptok * sh.ks_tok + ch];
    const int pm = real ? inline_mod(c.inl, b, ptok) : 0;
    if (pr < b_pad) lds_piv[pr * (NCH + 1) + ch] = v;
    float ss = chunk_sumsq<BF16>(v);
#pragma unroll
    for (int o = NCH / 2; o >= 1; o >>= 1) ss += __shfl_xor(ss, o, 64);
    if (ch == 0 && pr < b_pad) {
      const bool ok = real && !(__uint_as_float(lds_keys[ptok]) > s.tau);
      lds_w[pr] = inverse_norm(ss);
      lds_bias[pr] = ok && pm == 0 ? 0.f : -INFINITY;
      lds_bias[b_pad + pr] = ok && pm == 1 ? 0.f : -INFINITY;
    }
  }
  __syncthreads();

  const int nblk = b_pad >> 5;
  int dropped = 0;
  for (; t < ntiles; t += kF2Waves) {
    const int tok = t * 32 + n;
    const int tc = min(tok, L - 1);
    const int cur = lds_assign[tc];
    const float *bias = lds_bias + (inline_mod(c.inl, b, tc) ? b_pad : 0);
    // (the next tile's rows on their way meanwhile, where there are registers for two)
    constexpr bool kNext = THREADS == 256 || BF16;
    uint4 nxt[NF];
    if (kNext && t + kF2Waves < ntiles) {
      const uint4 *row = K + (long long)min((t + kF2Waves) * 32 + n, L - 1) * sh.ks_tok + half;
#pragma unroll
      for (int f = 0; f < NF; ++f) nxt[f] = row[2 * f];
    }
    float best = -INFINITY;
    int best_slot = -1;
    for (int pb = 0; pb < nblk; ++pb) {
      f32x16_t acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0.f;
      const uint4 *prow = lds_piv + (pb * 32 + n) * (NCH + 1) + half;
#pragma unroll
      for (int f = 0; f < NF; ++f) mma_chunk<BF16>(acc, prow[2 * f], kf[f]);  // [pivot][token]
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int pr = pb * 32 + acc_row(i, half);
        const float u = fmaf(acc[i], lds_w[pr], bias[pr]);
        if (u > best) { best = u; best_slot = pr; }
      }
    }
    const float ob = __shfl_xor(best, 32, 64);
    const int os = __shfl_xor(best_slot, 32, 64);
    if (ob > best || (ob == best && (unsigned)os < (unsigned)best_slot)) { best = ob; best_slot = os; }
    if (half == 0 && tok < L) {
      assign[tok] = cur == -2 ? best_slot : cur;  // a pivot keeps its own slot
      dropped += cur == -2 && best_slot < 0;
    }
    if (t + kF2Waves < ntiles) {
      const uint4 *row = K + (long long)min((t + kF2Waves) * 32 + n, L - 1) * sh.ks_tok + half;
#pragma unroll
      for (int f = 0; f < NF; ++f) kf[f] = kNext ? nxt[f] : row[2 * f];
    }
  }
  dropped = wave_sum_int(dropped);
  if (lane == 0 && dropped) atomicAdd(&sh_dropped, dropped);
  __syncthreads();
  if (threadIdx.x == 0) c.n_dropped[unit * sh.batch + b] = sh_dropped;
}

template <bool BF16, int D, int THREADS>
__global__ __launch_bounds__(THREADS) void unit_match_kernel(Ctx c, int b_pad) {
  extern __shared__ __align__(16) char lds_dyn[];
  const int b = rotated_block_x(), gkv = blockIdx.y, l = blockIdx.z + c.layer0;
  // unit_plan_kernel has matched the unit as a cross-modal layer does
  if (!unit_flow(c, b, gkv, l)) unit_intra_match_body<BF16, D, THREADS>(c, b_pad, lds_dyn, b, gkv, l);
}

// ============================ merge =========================================================
// Merge of one unit per workgroup (unit_merge_core.h).
// FLOW: the workgroup first settles its layer's strategy and, in an intra-modal layer, matches its
// unit again (what unit_match_kernel does), so that plan and merge take two launches, not three.
// bf16, 256 threads: four waves per SIMD, so that four workgroups share a compute unit (the weighted variant took 131 registers, matrix accumulators among
// them, and three did: 1024 units x 256 tokens 80 us a call, 69 with 116; x 541 142 and 128).
template <bool BF16, int D, int THREADS, int ROUNDS, int U, bool FLOW, bool WEIGHTED, bool DIVIDE>
__global__ __launch_bounds__(THREADS, BF16 || THREADS > 256 ? 4 : 1) void unit_merge_kernel(Ctx c, int maxB, int maxE, int b_pad) {
  extern __shared__ __align__(16) int lds_i[];
  __shared__ long long lds_wave[THREADS / 64 + 1];
  __shared__ int sh_next;
  const Shape &sh = c.sh;
  const int b = rotated_block_x(), gkv = blockIdx.y, l = blockIdx.z + c.layer0;
  const SeqInfo s = inline_seq(c.inl, b);
  const long long unit = (long long)l * sh.Hkv + gkv;
  auto settle = [&] {
    if constexpr (FLOW) {
      if (unit_flow(c, b, gkv, l)) return false;
      unit_intra_match_body<BF16, D, THREADS>(c, b_pad, reinterpret_cast<char *>(lds_i), b, gkv, l);
      __syncthreads();  // the assignment written above is read below; the LDS block changes hands
      return true;
    }
    return false;
  };
  unit_merge_body<BF16, D, THREADS, ROUNDS, U, WEIGHTED, DIVIDE>(c, s, unit, l, gkv, c.assign + unit * sh.T + s.tok_off, c.kept_idx + unit * sh.SB + s.kept_off,
                                                 lds_i, maxB, maxE, lds_wave, &sh_next, settle);
}

// ---- dispatch --------------------------------------------------------------------------------
int unit_nch(const Shape &sh) { return sh.d * (sh.bf16 ? 2 : 4) / 16; }  // 16-byte chunks of a row

size_t plan_lds_bytes(const Shape &sh, int b_pad) {
  return (size_t)plan_lds_layout(sh.R_pad, b_pad, unit_nch(sh)).total_bytes;
}

template <bool BF16, int D, int RB, int NT, int WAVES, bool PAIR = false, Operand KEYS = kPlain>
hipError_t launch_plan_k(const Ctx &c, int b_pad, size_t lds) {
  hipError_t e = allow_full_lds<unit_plan_kernel<BF16, D, RB, NT, WAVES, PAIR, KEYS>>();
  if (e != hipSuccess) return e;
  ProfScope ps(c.stream, KID_UNIT_PLAN);
  unit_plan_kernel<BF16, D, RB, NT, WAVES, PAIR, KEYS><<<dim3(c.sh.batch, c.sh.Hkv, c.layers), WAVES * 64, lds, c.stream>>>(c, b_pad);
  return hipGetLastError();
}

// fp32, one key tile a wave: whether its products are by the bf16 matrix cores, the keys split once.  That is quicker for a workgroup, but its registers leave a
// compute unit one workgroup of twelve waves in the place of two (64 channels), one of eight in the place of two (128): with more units than
// compute units the second one is worth more where a workgroup has much to wait for and little to multiply, up to 32 query rows.  Whole calls, fp32
// instructions -> split, us: 64 channels, 9 to 12 tiles: 256 units x 384 tokens 43.2 -> 39.7, 288 x 300 52.2 -> 53.1, 512 x 384 69.9 -> 71.4, 1024 x 300 107 -> 112,
// 2048 x 384 259 -> 271; 64 rows: 512 x 384 84.3 -> 81.7, 1024 x 300 133 -> 134; up to 8 tiles: 288 x 230 41.5 -> 36.2, 1024 x 230 81.8 -> 74.1.  128 channels, up to 8
// tiles: 512 x 230 77.7 -> 78.5, 1024 x 230 147 -> 158, 2048 x 230 298 -> 321, x 100 221 -> 225, 768 x 100 91.3 -> 88.4, 384 x 100 57.7 -> 56.9; 64 rows: 1024 x 230 216 -> 196; 9 to 12
// tiles (one workgroup either way): 1024 x 300 226 -> 205.
template <int D>
bool plan_splits_keys(const Ctx &c, int tiles) {
  const long long units = (long long)c.sh.batch * c.sh.Hkv * c.layers;
  return D == 64 ? tiles <= 8 || units <= 256 : tiles > 8 || units * tiles < 4096;
}

template <bool BF16, int D, int RB, Operand KEYS>
hipError_t launch_plan_one(const Ctx &c, int tiles, int b_pad, size_t lds) {  // one key tile a wave
  return tiles <= 8 ? launch_plan_k<BF16, D, RB, 1, 8, false, KEYS>(c, b_pad, lds) : launch_plan_k<BF16, D, RB, 1, 12, false, KEYS>(c, b_pad, lds);
}

template <bool BF16, int D, int RB>
hipError_t launch_f1(const Ctx &c) {
  const int b_pad = (c.sh.maxB + 31) / 32 * 32;
  const size_t lds = plan_lds_bytes(c.sh, b_pad);
  // Key tiles per wave and waves per workgroup: the unit's keys must fit the registers of one
  // workgroup, and twelve waves with two tiles each need fewer registers per wave (three waves per
  // SIMD) than eight waves with three.
  const int tiles = (c.sh.maxL + 31) / 32;
  // More units than compute units: eight waves of at most 128 registers, so that two workgroups share a compute unit and
  // one's barriers and trips to memory fall into the other's work.  Two tiles per wave fit; a third one is read from the L2 in
  // each of its passes (holding it too took 50 spilled registers and 108 us for 1024 units of 675 tokens; 84 with twelve waves
  // alone on the compute unit, 81 like this; 500 tokens: 130 us a pass with one workgroup per compute unit, 110 with two).
  if constexpr (Cfg<BF16, D>::NCH <= 16)
    if ((long long)c.sh.batch * c.sh.Hkv * c.layers > 256 && 2 * lds <= kLdsBytes - 16 * 1024) {
      if (tiles > 12 && tiles <= 16) return launch_plan_k<BF16, D, RB, 2, 8, true>(c, b_pad, lds);
      if (tiles > 16 && tiles <= 24) return launch_plan_k<BF16, D, RB, 3, 8, true>(c, b_pad, lds);
    }
  if (tiles <= 12) {
    if constexpr (BF16) return launch_plan_one<BF16, D, RB, kPlain>(c, tiles, b_pad, lds);
    else if constexpr (RB > 1) return launch_plan_one<BF16, D, RB, kSplitOnce>(c, tiles, b_pad, lds);
    else return plan_splits_keys<D>(c, tiles) ? launch_plan_one<BF16, D, RB, kSplitOnce>(c, tiles, b_pad, lds) : launch_plan_one<BF16, D, RB, kPlain>(c, tiles, b_pad, lds);
  }
  if (tiles <= 16 || Cfg<BF16, D>::NCH > 16) return launch_plan_k<BF16, D, RB, 2, 8>(c, b_pad, lds);
  if constexpr (Cfg<BF16, D>::NCH <= 16) {
    if (tiles <= 24) return launch_plan_k<BF16, D, RB, 2, 12>(c, b_pad, lds);
    return launch_plan_k<BF16, D, RB, 4, 8>(c, b_pad, lds);
  }
}

size_t match_lds_bytes(const Shape &sh, int b_pad) {
  return (size_t)match_lds_layout(b_pad, unit_nch(sh), sh.maxL).total_bytes;
}

template <bool BF16, int D, int THREADS>
hipError_t launch_f2t(const Ctx &c) {
  const int b_pad = (c.sh.maxB + 31) / 32 * 32;
  const size_t lds = match_lds_bytes(c.sh, b_pad);
  hipError_t e = allow_full_lds<unit_match_kernel<BF16, D, THREADS>>();
  if (e != hipSuccess) return e;
  ProfScope ps(c.stream, KID_UNIT_MATCH);
  unit_match_kernel<BF16, D, THREADS><<<dim3(c.sh.batch, c.sh.Hkv, c.layers), THREADS, lds, c.stream>>>(c, b_pad);
  return hipGetLastError();
}

// Threads of the match and merge workgroups.  Up to two units per compute unit eight waves each, which split a unit's trips to memory and its
// intra-modal match among them; more units keep a compute unit busy in fours of four waves but for long ones.  One call, four -> eight waves,
// us: 32 units x 220 tokens 29.6 -> 24.8; 128 x 675, intra-modal in half of the layers, 41.1 -> 36.5; 512 x 675 80.9 -> 77.2; 544 x 330 65.6 and
// 68.5, x 675 107 and 111, x 1000 198 -> 181; 1024 x 450 97.7 and 100.8, x 675 162.6 and 161.4, x 1000 296 -> 285; 4 fp32 units x 330 34.9 -> 32.1
// (sixteen waves: 25.3, 37.4, 87.6, .., 32.2).  Long ones of equal length with up to 128 pivots have little to share: between one and three rounds of the chip eight
// waves lose what they gain elsewhere, the more where layers are intra-modal (four -> eight, half of the layers: 576 x 850 tokens 153.5 -> 143.5, 768 x 924 186.7 -> 190.3,
// 640 x 1000 209 -> 220, 1024 x 850 224 -> 240, x 1000 285 -> 280, 2048 x 850 461 -> 440; 90 tokens kept of 850 in a cross-modal model 768 x 156.5 -> 157.3; 170 kept 195.7 -> 180.3).  Of 90
// batches of long and short sequences eight waves are quicker in 70, by up to 14 %, and at most 3 % slower (the rule takes the longest: the mean length does not tell them
// apart).
int merge_threads(const Shape &sh) {
  const long long units = (long long)sh.batch * sh.Hkv * sh.n_layers;
  if (units <= 512) return 512;
  const bool equal = (long long)sh.maxL * sh.batch == sh.T;
  return sh.maxL > 768 && (!equal || units <= 576 || units >= 1536 || (units >= 1024 && sh.maxL > 960) || sh.maxB > 128) ? 512 : 256;
}

template <bool BF16, int D>
hipError_t launch_f2(const Ctx &c) {
  const int t = merge_threads(c.sh);
  return t == 512 ? launch_f2t<BF16, D, 512>(c) : launch_f2t<BF16, D, 256>(c);
}

template <bool BF16, int D, int THREADS, int ROUNDS, int U, bool FLOW, bool WEIGHTED, bool DIVIDE>
hipError_t launch_f3w(const Ctx &c) {
  const int b_pad = (c.sh.maxB + 31) / 32 * 32;
  size_t lds = (size_t)merge_lds_layout(c.sh.maxB, c.sh.maxE, D, THREADS).total_bytes;
  if (FLOW && match_lds_bytes(c.sh, b_pad) > lds) lds = match_lds_bytes(c.sh, b_pad);
  hipError_t e = allow_full_lds<unit_merge_kernel<BF16, D, THREADS, ROUNDS, U, FLOW, WEIGHTED, DIVIDE>>();
  if (e != hipSuccess) return e;
  ProfScope ps(c.stream, FLOW ? KID_UNIT_FLOW_MERGE : KID_UNIT_MERGE);
  unit_merge_kernel<BF16, D, THREADS, ROUNDS, U, FLOW, WEIGHTED, DIVIDE><<<dim3(c.sh.batch, c.sh.Hkv, c.layers), THREADS, lds, c.stream>>>(
      c, c.sh.maxB, c.sh.maxE, b_pad);
  return hipGetLastError();
}

// Rows in flight per lane group: eight, or four in the weighted variant, whose cosines need every row of a trip in registers.  (While the
// rows past a task's end were read again, two were best with four workgroups on every compute unit, 80 us against 102 for 1024 units of
// 675 tokens.  Now they cost no traffic: a call with these units 164.5 us as it was, 162.5 with two, 161.9 with four, 161.1 with eight; 4
// units x 320 tokens, eight in both, 36.4 -> 34.9.)
// Plans of the generic kernels: eight waves however many units there are (one call, eight -> four, us: 144 units x 900 tokens 89 -> 103, 512 x 330 106 -> 109; from 1024 short
// ones on four are quicker, 1024 x 330 180 -> 174, 2048 x 150 256 -> 238, and so far not built).
template <bool BF16, int D, bool FLOW, bool WEIGHTED>
hipError_t launch_f3(const Ctx &c) {
  constexpr int U = WEIGHTED ? 4 : 8;
  if constexpr (!FLOW)
    if (!c.sh.unit_path)
      return c.sh.maxL <= 1024 ? launch_f3w<BF16, D, 512, 2, U, FLOW, WEIGHTED, true>(c) : launch_f3w<BF16, D, 512, 4, U, FLOW, WEIGHTED, true>(c);
  return merge_threads(c.sh) == 512 ? launch_f3w<BF16, D, 512, 2, U, FLOW, WEIGHTED, false>(c) : launch_f3w<BF16, D, 256, 4, U, FLOW, WEIGHTED, false>(c);
}

}  // namespace

// Longest sequence that a workgroup takes whole.  Rows of 512 bytes leave room for two tiles of 32 keys per wave.
// fp32 contractions run at a sixteenth of the bf16 rate and bind the workgroup: the generic kernels spread a unit over several
// of them, so where there are fewer units than compute units the long ones go there.  One call, generic -> unit path, us: 64 channels,
// 4 units: 512 tokens 57 -> 53, 544 57 -> 64, 1024 66 -> 112; 64 units: 544 63 -> 65; 112 units: 768 90 -> 80; 128 units: 1024
// 105 -> 117; 192 units: 1024 154 -> 120.  128 channels, 4 units: 384 tokens 71 -> 62, 400 71 -> 73, 512 75 -> 86; 112 units: 512 105 -> 91.
static int unit_max_tokens(const Shape &sh) {
  const bool wide = unit_nch(sh) > 16;
  const long long wgs = (long long)sh.batch * sh.Hkv * sh.n_layers;
  if (sh.bf16 || wgs >= 160) return wide ? 512 : 1024;
  if (wgs >= 96) return wide ? 512 : 768;
  return wide ? 384 : 512;
}

bool unit_path_fits(const Shape &sh) {
  // A workgroup matches its whole unit: with fewer units than half the compute units and long lists the generic kernels, which spread a unit over
  // several workgroups, are quicker.  One call, generic -> unit path, us: 128 channels, 4 units: 700 tokens, 140 pivots 50.0 -> 50.9, 1000, 200 54.6 -> 66.1; 56 units:
  // 1000, 200 64.3 -> 74.6; 112: 1000, 250 75.6 -> 79.8, 700, 140 62.7 -> 55.4; 64 channels, 16 units: 1000, 250 50.9 -> 57.9, 700, 140 45.4 -> 44.9.
  if (sh.bf16 && (long long)sh.batch * sh.Hkv * sh.n_layers < 128 && (long long)sh.maxE * sh.maxB > 120000) return false;
  if (sh.maxL > unit_max_tokens(sh) || sh.R_pad > 64 || sh.maxB > 256 || sh.Hq > 4096) return false;
  if (sh.batch > kInlineSeqs || sh.n_spans > kInlineSpans) return false;  // metadata must fit the kernel arguments
  if (sh.ks_tok * 16 * 1024 >= (1ll << 32)) return false;  // the merge addresses a sequence's rows with 32-bit offsets
  const int b_pad = (sh.maxB + 31) / 32 * 32;
  if (match_lds_bytes(sh, b_pad) > 150 * 1024 || plan_lds_bytes(sh, b_pad) > 150 * 1024) return false;
  if ((size_t)merge_lds_layout(sh.maxB, sh.maxE, sh.d, 512).total_bytes > 150 * 1024) return false;
  return true;
}

// Whether a plan of the generic kernels is merged by one workgroup per unit: one launch in the place of two, the grouping and the
// tasks.  Its workgroup moves a unit's rows alone, so units have to fill half of the chip with short sequences; longer ones three quarters to
// all of it, equal.  Beyond one round the first 64 units of the next lose (288 x 2000 tokens 231 -> 242, 544 x 1400 319 -> 330) and a filled one wins, 64 channels
// most (512 x 1065 of 128 channels 175 -> 168, of 64 123 -> 110, 1024 x 1065 of 64 225 -> 201): 256 is not where the gain ends, but 512 and 520 units are what the tests of
// the grouping kernel beside the split and match are made of.  One call, separate kernels -> one, us: 28/4 heads, 64 units x 300
// tokens 46.6 -> 48.4; 136 x 900 93.7 -> 84.3; 256 x 800 113 -> 98.7; 336 x 900 194 -> 162; 768 x 900 324 -> 282; 112 x 1200, 240 pivots 93.6 -> 95.7; 168 x 1700, 340 pivots
// 164 -> 167, 224 x 1700 197 -> 191; 320 x 1700 248 -> 252; 336 unequal x 1700 199 -> 202; 256 x 2500 291 -> 285, 512 x 3200 622 -> 624; fp32 256 x 700 197 -> 182.
bool unit_merge_fits(const Shape &sh) {
  const long long units = (long long)sh.batch * sh.Hkv * sh.n_layers;
  if (sh.batch > kInlineSeqs || !sh.rows32 || sh.maxB > 512 || sh.maxL > 2048 || units < 128) return false;
  const size_t lds = (size_t)merge_lds_layout(sh.maxB, sh.maxE, sh.d, 512).total_bytes;
  return lds <= 150 * 1024 && (sh.maxL <= 1024 || (units >= 192 && units <= 256 && (long long)sh.maxL * sh.batch == sh.T));
}

namespace {

template <bool BF16, int D, bool FLOW>
hipError_t launch_unit_merge_f(const Ctx &c) {
  return c.sh.weighted_merge ? launch_f3<BF16, D, FLOW, true>(c) : launch_f3<BF16, D, FLOW, false>(c);
}

template <bool BF16, int D>
hipError_t launch_unit_merge_t(const Ctx &c, bool with_flow) {
  return with_flow ? launch_unit_merge_f<BF16, D, true>(c) : launch_unit_merge_f<BF16, D, false>(c);
}

template <bool BF16, int D>
hipError_t launch_unit_plan_t(const Ctx &c) {
  return c.sh.R_pad == 32 ? launch_f1<BF16, D, 1>(c) : launch_f1<BF16, D, 2>(c);
}

}  // namespace

hipError_t launch_unit_flow_match(const Ctx &c) {
  if (c.sh.bf16) return c.sh.d == 128 ? launch_f2<true, 128>(c) : launch_f2<true, 64>(c);
  return c.sh.d == 128 ? launch_f2<false, 128>(c) : launch_f2<false, 64>(c);
}

hipError_t launch_unit_plan(const Ctx &c, bool with_flow) {  // score + select + cross-modal match, then flow + intra-modal layers
  hipError_t e;
  if (c.sh.bf16) e = c.sh.d == 128 ? launch_unit_plan_t<true, 128>(c) : launch_unit_plan_t<true, 64>(c);
  else e = c.sh.d == 128 ? launch_unit_plan_t<false, 128>(c) : launch_unit_plan_t<false, 64>(c);
  if (e != hipSuccess || !with_flow) return e;
  return launch_unit_flow_match(c);
}

// with_flow: the launch also settles the layer strategies and rematches the intra-modal layers
// (then it takes the place of launch_unit_flow_match + launch_unit_merge after the plan kernel)
hipError_t launch_unit_merge(const Ctx &c, bool with_flow) {
  if (c.sh.bf16) return c.sh.d == 128 ? launch_unit_merge_t<true, 128>(c, with_flow) : launch_unit_merge_t<true, 64>(c, with_flow);
  return c.sh.d == 128 ? launch_unit_merge_t<false, 128>(c, with_flow) : launch_unit_merge_t<false, 64>(c, with_flow);
}

}  // namespace flowmm
