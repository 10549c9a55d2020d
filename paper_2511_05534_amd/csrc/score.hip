// Step "score": attention of the proxy (window) queries over all cached keys, reduced to the
// proxy importance of every key and to each query head's cross-modal attention mass
// (FlowMM, Information Flow Guided Merging: importance equation and the A_{v->t}, A_{t->v}
// sums; attention as in the Preliminary section).
//
// Three sets of kernels: one workgroup takes a whole short sequence (score_resident), in bf16 the query rows stay
// in registers while the keys stream through LDS (score_stream_*), and everything else (fp32, more than 256 query rows) as
// follows.
// The logits tile of a workgroup never leaves registers.  Keys are split across workgroups,
// so the softmax needs every row's global (max, sum): pass 1 writes those per run of tiles, pass 2
// folds them per row into one offset c = max + log2(sum), recomputes the tile's
// logits and reduces exp2(logit - c) over the query rows.  Both heavy passes read K once,
// straight from HBM into MFMA operand registers (one 16-byte chunk per lane and k step, 32*KS
// keys per wave); the query rows of the (sequence, kv head, layer) arrive in LDS by direct
// global->LDS loads and every fragment read from there feeds KS matrix instructions.
// Only the tiles that reach into the window (or past the end of the sequence) pay for the
// causal mask; only sequences whose window holds image tokens pay for per-row modality weights.
#include <cfloat>

#include "device_common.h"
#include "kernels.h"
#include "profile.h"
#include "score_core.h"
#include "select_core.h"

namespace flowmm {

namespace {

constexpr int kThreads = kScoreWaves * 64;

size_t score_resident_lds(const Shape &sh, int waves) {
  const int nch = sh.d * (sh.bf16 ? 2 : 4) / 16;
  return (size_t)sh.R_pad * (nch + 1) * 16 + ((size_t)(waves + 3) * sh.R_pad + waves) * sizeof(float);
}

struct TileCtx {
  int b, tile, x, gkv, l, wave, lane, n, half, key0;  // key0: first key of this wave in the current tile
  int tile_end;                                       // the run covers tiles [tile, tile_end) of sequence b
  bool masked;                                        // some key of the current tile is hidden from some window row
  SeqInfo s;
};

// workgroups of the kernels over tiles or runs of tiles
__host__ __device__ __forceinline__ int tiles_grid(const Shape &sh) { return (sh.n_layers * sh.Hkv * sh.tiles_score + 7) / 8 * 8; }

// Returns false for the padding workgroups.
template <int TILE>
__device__ __forceinline__ bool tile_ctx(const Ctx &c, ScalarInts meta, TileCtx &t) {
  const Shape &sh = c.sh;
  int unit;
  if (!xcd_share(sh.n_layers * sh.Hkv * sh.tiles_score, sh.tiles_score, unit, t.x)) return false;
  t.l = unit / sh.Hkv;
  t.gkv = unit - t.l * sh.Hkv;
  const ScalarInts cu = meta + meta[MW_OFF_CU_SCORE];
  t.b = find_seq(cu, meta[MW_BATCH], t.x);
  t.s = load_seq(meta, t.b);
  t.tile = (t.x - cu[t.b]) * sh.score_tpw;
  t.tile_end = min(t.tile + sh.score_tpw, (t.s.L + TILE - 1) / TILE);
  t.wave = threadIdx.x >> 6;
  t.lane = threadIdx.x & 63;
  t.n = t.lane & 31;
  t.half = t.lane >> 5;
  t.key0 = t.tile * TILE + t.wave * (TILE / kScoreWaves);
  t.masked = (t.tile + 1) * TILE > t.s.L - sh.W;
  return true;
}

// position the context on tile `tile` of the run
template <int TILE>
__device__ __forceinline__ void set_tile(const Ctx &c, TileCtx &t, int tile) {
  t.tile = tile;
  t.key0 = tile * TILE + t.wave * (TILE / kScoreWaves);
  t.masked = (tile + 1) * TILE > t.s.L - c.sh.W;
}

// Request the R_pad query rows of this (sequence, layer, kv head) into LDS, row stride NCH+1
// chunks (the odd stride keeps the 16-byte fragment reads of 16 consecutive rows on distinct
// banks).  The heads' windows lie next to each other, W rows each (four heads of 16 proxy tokens are two blocks of 32 rows, not four);
// rows past the last one, and the padding chunk of every row, are zeros.
template <bool BF16, int D, int THREADS = kThreads>
__device__ __forceinline__ void stage_queries(const Ctx &c, const TileCtx &t, uint4 *ldsq) {
  constexpr int NCH = Cfg<BF16, D>::NCH, RS = NCH + 1;
  const Shape &sh = c.sh;
  const uint4 *Q = reinterpret_cast<const uint4 *>(c.Q) + (long long)t.l * sh.qs_layer +
                   (long long)(t.gkv * sh.G) * sh.qs_head + (long long)(t.b * sh.W) * sh.qs_tok;
  const int total = sh.R_pad * RS;
  // chunk q of the LDS image is chunk ch of row r of head g; q advances by the workgroup size per
  // trip, so (g, r, ch) are carried along instead of being divided out again
  constexpr int kRowStep = THREADS / RS, kChStep = THREADS % RS;
  int q = t.wave * 64 + t.lane;
  int row = q / RS, ch = q - row * RS;
  int g = row / sh.W, r = row - g * sh.W;
  for (int q0 = t.wave * 64; q0 < total; q0 += THREADS) {
    if (q0 + t.lane < total) {
      if (g < sh.G && ch < NCH)
        load_to_lds<16>(Q, (unsigned)(g * sh.qs_head + r * sh.qs_tok + ch) * 16u, ldsq + q0);
      else
        ldsq[q0 + t.lane] = make_uint4(0, 0, 0, 0);  // padding rows and the padding chunk of every row
    }
    ch += kChStep;
    r += kRowStep;
    if (ch >= RS) { ch -= RS; ++r; }
    while (r >= sh.W) { r -= sh.W; ++g; }
  }
}

// this lane's first fragment of its key of group `sub` (the last key again past the end)
__device__ __forceinline__ const uint4 *key_row(const Ctx &c, const TileCtx &t, int sub) {
  const Shape &sh = c.sh;
  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)t.l * sh.ks_layer +
                   (long long)t.gkv * sh.ks_head;
  return K + (long long)(t.s.tok_off + min(t.key0 + sub * 32 + t.n, t.s.L - 1)) * sh.ks_tok + t.half;
}

template <bool BF16, int D, int KS>
__device__ __forceinline__ void load_keys(const Ctx &c, const TileCtx &t, uint4 (&kf)[KS][Cfg<BF16, D>::NF]) {
#pragma unroll
  for (int sub = 0; sub < KS; ++sub) {
    const uint4 *row = key_row(c, t, sub);
#pragma unroll
    for (int f = 0; f < Cfg<BF16, D>::NF; ++f) kf[sub][f] = row[2 * f];
  }
}

// The keys as matrix operands.  fp32: split once for all blocks of query rows, but for 128 channels in sixteen waves, which have no registers for it.
template <bool BF16, int D, int WAVES>
constexpr Operand key_operand() { return !BF16 && (D == 64 || WAVES == 8) ? kSplitOnce : kPlain; }
// waves per SIMD that the registers are shared among
template <bool BF16, int D, int WAVES>
constexpr int score_waves_per_simd() { return !BF16 && D == 128 && WAVES == 8 ? 2 : 4; }
template <bool BF16, int D, int KS, int WAVES>
using KeyRegs = RowOperand<Cfg<BF16, D>::NF, key_operand<BF16, D, WAVES>()>[KS];

// The products of one block of 32 query rows (this lane's first fragment at qrow) with this wave's keys; see block_products.
template <bool BF16, int D, int KS, bool KEYS_AS_ROWS, int AHEAD, class Keys>
__device__ __forceinline__ void tile_products(const Ctx &c, const TileCtx &t, f32x16_t (&acc)[KS], Keys &kf, uint4 (&pf)[AHEAD], const char *qrow, bool more) {
  if constexpr (BF16) block_products<D, KS, KEYS_AS_ROWS, AHEAD>(acc, kf, pf, qrow, more);
  else f32_products<KEYS_AS_ROWS>(acc, kf, [&](int f) { return *reinterpret_cast<const uint4 *>(qrow + 32 * f); }, [&](int sub, int f) { return key_row(c, t, sub)[2 * f]; });
}

// last key that a query row may see, -1 for the rows past the last one
__device__ __forceinline__ int row_limit(const Shape &sh, const SeqInfo &s, int row) {
  return row < sh.G * sh.W ? s.L - sh.W + window_row(sh, row) : -1;
}

// ---- pass 1: per-tile row statistics ---------------------------------------------------
template <bool BF16, int D, int KS, int WAVES, bool MASKED>
__device__ __forceinline__ void stats_body(const Ctx &c, const TileCtx &t, KeyRegs<BF16, D, KS, WAVES> &kf,
                                           const uint4 *ldsq, float *lds_stats) {
  constexpr int NF = Cfg<BF16, D>::NF, RS = Cfg<BF16, D>::NCH + 1;
  constexpr int AHEAD = NF < 2 ? NF : 2;
  const Shape &sh = c.sh;
  const int RB = sh.R_pad >> 5;
  const float cl = sh.scale_log2e;
  const char *qbase = reinterpret_cast<const char *>(ldsq) + (t.n * RS + t.half) * 16;
  uint4 pf[AHEAD];
  if constexpr (BF16) {
#pragma unroll
    for (int f = 0; f < AHEAD; ++f) pf[f] = *reinterpret_cast<const uint4 *>(qbase + 32 * f);
  }
  for (int rb = 0; rb < RB; ++rb) {
    f32x16_t acc[KS];
    tile_products<BF16, D, KS, true, AHEAD>(c, t, acc, kf, pf, qbase + rb * (32 * RS * 16), rb + 1 < RB);  // [key][query row]
    const int row = rb * 32 + t.n;
    float m = -INFINITY, z = 0.f;
    if constexpr (MASKED) {
      const int limit = row_limit(sh, t.s, row);
#pragma unroll
      for (int sub = 0; sub < KS; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = t.key0 + sub * 32 + acc_row(i, t.half);
          acc[sub][i] = key <= limit ? acc[sub][i] : -INFINITY;
          m = fmaxf(m, acc[sub][i]);
        }
      if (m > -INFINITY) {
        const float mc = m * cl;
#pragma unroll
        for (int sub = 0; sub < KS; ++sub)
#pragma unroll
          for (int i = 0; i < 16; ++i) z += fast_exp2(fmaf(acc[sub][i], cl, -mc));
      }
      m *= cl;
    } else {
#pragma unroll
      for (int sub = 0; sub < KS; ++sub)
#pragma unroll
        for (int i = 0; i < 16; i += 2) m = fmaxf(fmaxf(m, acc[sub][i]), acc[sub][i + 1]);
      m *= cl;  // cl > 0: the largest logit is the largest product
#pragma unroll
      for (int sub = 0; sub < KS; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) z += fast_exp2(fmaf(acc[sub][i], cl, -m));
    }
    const float m2 = __shfl_xor(m, 32, 64), z2 = __shfl_xor(z, 32, 64);
    stat_combine(m, z, m2, z2);
    // log2 of the row's sum of 2^logit over this wave's keys so far in the run: the pair (that, 1)
    // stands for (m, z); the slot belongs to this lane, earlier tiles of the run left their sum there
    if (t.half == 0) {
      float *slot = lds_stats + t.wave * sh.R_pad + row;
      float m0 = *slot, z0 = m0 == -INFINITY ? 0.f : 1.f;
      stat_combine(m0, z0, m, z);
      *slot = z0 > 0.f ? m0 + __builtin_amdgcn_logf(z0) : -INFINITY;
    }
  }
}

// RUN: the workgroup may have several tiles (a loop around the tile costs a few registers that the
// one-tile kernel, which small workloads get, does not have to spill)
template <bool BF16, int D, bool RUN>
__global__ __launch_bounds__(kThreads, (score_waves_per_simd<BF16, D, kScoreWaves>())) void score_stats_kernel(KernelArgs<Ctx> k) {
  const Ctx &c = k.a;
  constexpr int NCH = Cfg<BF16, D>::NCH, NF = Cfg<BF16, D>::NF, KS = score_subs(BF16);
  extern __shared__ uint4 lds[];
  const Shape &sh = c.sh;
  const ScalarInts meta = first_meta(k, c.meta);
  TileCtx t;
  if (const int own = tiles_grid(sh); (int)blockIdx.x >= own) return place_meta<kThreads>(c, meta, k.meta.n, blockIdx.x - own);
  if (!tile_ctx<score_tile_keys(BF16)>(c, meta, t)) return;
  uint4 *ldsq = lds;
  float *lds_stats = reinterpret_cast<float *>(lds + sh.R_pad * (NCH + 1));  // [waves][R_pad]
  uint4 kf[KS][NF];
  load_keys<BF16, D, KS>(c, t, kf);  // the long way first (HBM); the query rows come from L2
  stage_queries<BF16, D>(c, t, ldsq);
  for (int row = t.lane; row < sh.R_pad; row += 64) lds_stats[t.wave * sh.R_pad + row] = -INFINITY;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // the run's tiles one after the other on the same query rows; the workgroup that shares the compute
  // unit computes while this one waits for its next keys
  const int tile_end = RUN ? t.tile_end : t.tile + 1;
  for (int tile = t.tile; tile < tile_end; ++tile) {
    if (tile != t.tile) {
      set_tile<score_tile_keys(BF16)>(c, t, tile);
      load_keys<BF16, D, KS>(c, t, kf);
    }
    if (t.key0 < t.s.L) {  // waves past the end of the sequence have nothing to add
      KeyRegs<BF16, D, KS, kScoreWaves> keys;
#pragma unroll
      for (int sub = 0; sub < KS; ++sub) keys[sub].set(kf[sub]);
      if (t.masked) stats_body<BF16, D, KS, kScoreWaves, true>(c, t, keys, ldsq, lds_stats);
      else stats_body<BF16, D, KS, kScoreWaves, false>(c, t, keys, ldsq, lds_stats);
    }
  }
  __syncthreads();
  float2 *out = reinterpret_cast<float2 *>(c.part_stats) + ((long long)(t.l * sh.Hkv + t.gkv) * sh.tiles_score + t.x) * sh.R_pad;
  for (int row = threadIdx.x; row < sh.R_pad; row += kThreads) {
    float2 a = make_float2(lds_stats[row], 1.f);
    if (a.x == -INFINITY) a.y = 0.f;
#pragma unroll
    for (int w = 1; w < kScoreWaves; ++w) {
      const float o = lds_stats[w * sh.R_pad + row];
      stat_combine(a.x, a.y, o, o == -INFINITY ? 0.f : 1.f);
    }
    out[row] = a;
  }
}

// ---- pass 2: normalised probabilities reduced over the query rows ------------------------
// What the second pass knows of a query row, in LDS
struct RowTables {
  float *c;      // [R_pad] max + log2(sum): exp2(logit - c) is the normalised probability; +inf for padding rows, whose probability is 0
  float *img;    // [R_pad] 1 for an image token of the window
  int *limit;    // [R_pad] last key the row may see
  float *cross;  // [waves] cross-modal mass
};

template <bool BF16, int D, int KS, int WAVES, bool MASKED, bool WIN_IMG>
__device__ __forceinline__ void colsum_body(const Ctx &c, const TileCtx &t, KeyRegs<BF16, D, KS, WAVES> &kf,
                                            const int (&keymod)[KS], const uint4 *ldsq, const RowTables &rows, float (&colsum)[KS]) {
  constexpr int NF = Cfg<BF16, D>::NF, RS = Cfg<BF16, D>::NCH + 1;
  constexpr int AHEAD = 1;  // registers are short here: one fragment in flight
  const Shape &sh = c.sh;
  const int RB = sh.R_pad >> 5;
  const float cl = sh.scale_log2e;
  const char *qbase = reinterpret_cast<const char *>(ldsq) + (t.n * RS + t.half) * 16;
  uint4 pf[AHEAD];
  if constexpr (BF16) {
#pragma unroll
    for (int f = 0; f < AHEAD; ++f) pf[f] = *reinterpret_cast<const uint4 *>(qbase + 32 * f);
  }
  float cross_acc = 0.f;
  for (int rb = 0; rb < RB; ++rb) {
    f32x16_t acc[KS];
    tile_products<BF16, D, KS, false, AHEAD>(c, t, acc, kf, pf, qbase + rb * (32 * RS * 16), rb + 1 < RB);  // [query row][key]
    float bs[KS], bsi[KS];
#pragma unroll
    for (int sub = 0; sub < KS; ++sub) bs[sub] = bsi[sub] = 0.f;
    // rows 8g + 4 half + j of the block, j = 0..3 (the fences keep the compiler from fetching the
    // constants of all four groups up front: registers are short)
    const int row0 = rb * 32 + 4 * t.half;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 c4 = *reinterpret_cast<const float4 *>(rows.c + row0 + 8 * g);
      float4 w4 = make_float4(0.f, 0.f, 0.f, 0.f);
      int4 l4 = make_int4(0, 0, 0, 0);
      if constexpr (WIN_IMG) w4 = *reinterpret_cast<const float4 *>(rows.img + row0 + 8 * g);
      if constexpr (MASKED) l4 = *reinterpret_cast<const int4 *>(rows.limit + row0 + 8 * g);
      const float cr[4] = {c4.x, c4.y, c4.z, c4.w};
      const float wimg[4] = {w4.x, w4.y, w4.z, w4.w};
      const int lim[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
      for (int sub = 0; sub < KS; ++sub) {
        const int key = t.key0 + sub * 32 + t.n;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float p = fast_exp2(fmaf(acc[sub][4 * g + j], cl, -cr[j]));
          if constexpr (MASKED) p = key <= lim[j] ? p : 0.f;
          bs[sub] += p;
          if constexpr (WIN_IMG) bsi[sub] = fmaf(p, wimg[j], bsi[sub]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int sub = 0; sub < KS; ++sub) {
      colsum[sub] += bs[sub];
      // mass sent to the other modality: image keys seen by text rows, text keys by image rows
      if constexpr (WIN_IMG) cross_acc += keymod[sub] ? bs[sub] - bsi[sub] : bsi[sub];
      else cross_acc += keymod[sub] ? bs[sub] : 0.f;
    }
  }
  const float v = wave_sum(cross_acc);
  if (t.lane == 0) rows.cross[t.wave] += v;  // over the tiles of the run
}

template <bool BF16, int D, int KS, int WAVES>
__device__ __forceinline__ void colsum_any(const Ctx &c, const TileCtx &t, KeyRegs<BF16, D, KS, WAVES> &kf,
                                           const int (&keymod)[KS], const uint4 *ldsq, const RowTables &rows, float (&colsum)[KS]) {
  const bool win_img = t.s.win_has_img != 0;
  if (t.masked) {
    if (win_img) colsum_body<BF16, D, KS, WAVES, true, true>(c, t, kf, keymod, ldsq, rows, colsum);
    else colsum_body<BF16, D, KS, WAVES, true, false>(c, t, kf, keymod, ldsq, rows, colsum);
  } else {
    if (win_img) colsum_body<BF16, D, KS, WAVES, false, true>(c, t, kf, keymod, ldsq, rows, colsum);
    else colsum_body<BF16, D, KS, WAVES, false, false>(c, t, kf, keymod, ldsq, rows, colsum);
  }
}

// the tables but for c, and cleared sums
__device__ __forceinline__ void fill_row_tables(const Ctx &c, ScalarInts meta, int b, const SeqInfo &s, const RowTables &rows, int waves) {
  const Shape &sh = c.sh;
  for (int row = threadIdx.x; row < sh.R_pad; row += waves * 64) {
    const int limit = row_limit(sh, s, row);  // (a row's own position)
    rows.limit[row] = limit;
    rows.img[row] = limit >= 0 && late_modality(meta, b, s.L - sh.W, limit) ? 1.f : 0.f;
  }
  if ((int)threadIdx.x < waves) rows.cross[threadIdx.x] = 0.f;
}

// cross-modal mass of the kv head's rows
__device__ __forceinline__ void store_cross(const Ctx &c, const TileCtx &t, const RowTables &rows, int waves, int x) {
  if (threadIdx.x != 0) return;
  float v = 0.f;
  for (int w = 0; w < waves; ++w) v += rows.cross[w];
  c.cross_part[(long long)(t.l * c.sh.Hkv + t.gkv) * c.sh.tiles_score + x] = v;
}

// importances of this wave's keys: the two half-waves have seen disjoint query rows of the same keys
template <int KS>
__device__ __forceinline__ void store_importance(const Ctx &c, const TileCtx &t, const float (&colsum)[KS]) {
  const Shape &sh = c.sh;
  const float inv_rows = 1.0f / (float)(sh.G * sh.W);
  float *imp = c.importance + (long long)(t.l * sh.Hkv + t.gkv) * sh.T + t.s.tok_off;
#pragma unroll
  for (int sub = 0; sub < KS; ++sub) {
    const int key = t.key0 + sub * 32 + t.n;
    const float tot = colsum[sub] + __shfl_xor(colsum[sub], 32, 64);
    if (t.half == 0 && key < t.s.L) imp[key] = tot * inv_rows;
  }
}

template <bool BF16, int D, bool RUN>
__global__ __launch_bounds__(kThreads, (score_waves_per_simd<BF16, D, kScoreWaves>())) void score_colsum_kernel(Ctx c) {
  constexpr int NCH = Cfg<BF16, D>::NCH, NF = Cfg<BF16, D>::NF, KS = score_subs(BF16);
  extern __shared__ uint4 lds[];
  const Shape &sh = c.sh;
  TileCtx t;
  if (!tile_ctx<score_tile_keys(BF16)>(c, scalar_ints(c.meta), t)) return;
  uint4 *ldsq = lds;
  RowTables rows;
  rows.c = reinterpret_cast<float *>(lds + sh.R_pad * (NCH + 1));
  rows.img = rows.c + sh.R_pad;
  rows.limit = reinterpret_cast<int *>(rows.img + sh.R_pad);
  rows.cross = reinterpret_cast<float *>(rows.limit + sh.R_pad);

  uint4 kf[KS][NF];
  load_keys<BF16, D, KS>(c, t, kf);  // the long way first (HBM); the query rows come from L2
  stage_queries<BF16, D>(c, t, ldsq);
  {  // a row's statistics over the runs of its sequence, folded in the same order by every workgroup
    const int *cu = c.meta + c.meta[MW_OFF_CU_SCORE];
    const int x0 = cu[t.b], x1 = cu[t.b + 1];
    const float2 *in = reinterpret_cast<const float2 *>(c.part_stats) + (long long)(t.l * sh.Hkv + t.gkv) * sh.tiles_score * sh.R_pad;
    for (int row = threadIdx.x; row < sh.R_pad; row += kThreads) {
      float m = -INFINITY, z = 0.f;
      if (row < sh.G * sh.W) {
        for (int x = x0; x < x1; ++x) {
          const float2 o = in[(long long)x * sh.R_pad + row];
          stat_combine(m, z, o.x, o.y);
        }
      }
      rows.c[row] = z > 0.f ? m + __builtin_amdgcn_logf(z) : INFINITY;
    }
  }
  fill_row_tables(c, scalar_ints(c.meta), t.b, t.s, rows, kScoreWaves);
  const uint8_t *mod = c.mod + t.s.tok_off;
  int keymod[KS];
#pragma unroll
  for (int sub = 0; sub < KS; ++sub) {
    const int key = t.key0 + sub * 32 + t.n;
    keymod[sub] = mod[key < t.s.L ? key : t.s.L - 1];
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // the run's tiles one after the other on the same query rows (see score_stats_kernel)
  const int tile_end = RUN ? t.tile_end : t.tile + 1;
  for (int tile = t.tile; tile < tile_end; ++tile) {
    if (tile != t.tile) {
      set_tile<score_tile_keys(BF16)>(c, t, tile);
      load_keys<BF16, D, KS>(c, t, kf);
#pragma unroll
      for (int sub = 0; sub < KS; ++sub) {
        const int key = t.key0 + sub * 32 + t.n;
        keymod[sub] = mod[key < t.s.L ? key : t.s.L - 1];
      }
    }
    if (t.key0 >= t.s.L) continue;  // this wave's keys lie past the end of the sequence
    float colsum[KS];
#pragma unroll
    for (int sub = 0; sub < KS; ++sub) colsum[sub] = 0.f;
    KeyRegs<BF16, D, KS, kScoreWaves> keys;
#pragma unroll
    for (int sub = 0; sub < KS; ++sub) keys[sub].set(kf[sub]);
    colsum_any<BF16, D, KS, kScoreWaves>(c, t, keys, keymod, ldsq, rows, colsum);
    store_importance<KS>(c, t, colsum);
  }
  __syncthreads();
  store_cross(c, t, rows, kScoreWaves, t.x);
}

template <bool BF16, int D, bool RUN>
hipError_t launch_score_t(const Ctx &c, const int *words, int n_words) {
  constexpr int NCH = Cfg<BF16, D>::NCH;
  const Shape &sh = c.sh;
  const size_t q_bytes = (size_t)sh.R_pad * (NCH + 1) * 16;
  const size_t lds1 = q_bytes + (size_t)kScoreWaves * sh.R_pad * sizeof(float);
  const size_t lds3 = q_bytes + ((size_t)3 * sh.R_pad + kScoreWaves) * 4;
  hipError_t e;
  e = allow_full_lds<score_stats_kernel<BF16, D, RUN>>();
  if (e != hipSuccess) return e;
  e = allow_full_lds<score_colsum_kernel<BF16, D, RUN>>();
  if (e != hipSuccess) return e;
  if ((long long)sh.n_layers * sh.Hkv * sh.tiles_score + sh.n_spans > 0x7ffffff0LL) return hipErrorInvalidConfiguration;
  const unsigned grid = (unsigned)tiles_grid(sh);
  KernelArgs<Ctx> k;
  fill_kernel_args(k, c, words, n_words);
  {
    ProfScope ps(c.stream, KID_SCORE_STATS);
    score_stats_kernel<BF16, D, RUN><<<grid + (n_words ? sh.n_spans : 0), kThreads, lds1, c.stream>>>(k);
  }
  {
    ProfScope ps(c.stream, KID_SCORE_COLSUM);
    score_colsum_kernel<BF16, D, RUN><<<grid, kThreads, lds3, c.stream>>>(c);
  }
  return hipGetLastError();
}

// ---- bf16, up to four groups of 64 query rows: query rows in registers, keys streamed through LDS -------------
// A workgroup walks over a run of key tiles that arrive in LDS by direct global->LDS loads, double buffered
// (KeyTile).  Wave w holds 64 query rows (two groups of 32, as MFMA operands) and takes every KSPLIT-th block of 32 keys of
// a tile; a row group's waves together see all keys.  No wave waits for its own keys, the statistics of a row are
// two registers of the lane that owns it in the first pass, and the query rows are fetched once per run.
// Bound by the block loop: per 64 logits 16 cycles of matrix core and 12 to 13 of vector issue (v_exp_f32 8, multiply-add,
// add, half a maximum in the first pass), with the clock held down by the power limit.
// 256 units x 16384 keys x 256 rows: 338 + 5 + 340 us through the kernels above (statistics, fold, sums), 303 + 321 here;
// 112 units x 4096 keys x 224 rows: 48 + 5 + 49, here 42 + 43.  The second pass keeps the first one's orientation (a row's
// constant is then one register; with keys in lanes the constants of 64 rows come from LDS for every block, which filled its
// bandwidth: 395 us) and pays for it with the sum over lanes.
// Waves of a workgroup: eight, or four with up to 64 query rows, all of which each of them then holds (a block of keys each of a tile of four).
__host__ __device__ constexpr int stream_waves(int rows) { return rows <= 64 ? 4 : 8; }
// two workgroups fit a compute unit's LDS, of 64 channels four
template <int D, int WAVES>
constexpr int stream_waves_per_simd() { return WAVES == 4 && D == 128 ? 2 : 4; }

struct StreamCtx {
  int b, x, gkv, l, wave;
  int tile, tile_end;     // key tiles [tile, tile_end) of sequence b
  int ksplit, ks, rg;     // this wave: row group rg, key blocks ks, ks + ksplit, .. of a tile
  int rb0, nrb;           // its first block of 32 query rows, and how many (1 or 2)
  SeqInfo s;
};

template <int D, int WAVES>
__device__ __forceinline__ bool stream_ctx(const Ctx &c, ScalarInts meta, StreamCtx &t) {
  constexpr int KT = KeyTile<true, D>::kRows;
  const Shape &sh = c.sh;
  int unit;
  if (!xcd_share(sh.n_layers * sh.Hkv * sh.tiles_score, sh.tiles_score, unit, t.x)) return false;
  t.l = unit / sh.Hkv;
  t.gkv = unit - t.l * sh.Hkv;
  const ScalarInts cu = meta + meta[MW_OFF_CU_SCORE];
  t.b = find_seq(cu, meta[MW_BATCH], t.x);
  t.s = load_seq(meta, t.b);
  t.tile = (t.x - cu[t.b]) * sh.score_tpw;
  t.tile_end = min(t.tile + sh.score_tpw, (t.s.L + KT - 1) / KT);
  t.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = sh.R_pad >> 5;
  if constexpr (WAVES == 4) {
    t.ksplit = 4; t.rg = 0; t.ks = t.wave;
    t.rb0 = 0; t.nrb = rb;
  } else {
    // Two row groups of four waves each or four of two.  The blocks of 32 rows are dealt out evenly, the first groups get the ones that are left over
    // (waves w and w + 4 share a SIMD: with six blocks every SIMD has three at a time).
    t.ksplit = rb > 4 ? 2 : 4;
    const int groups = 8 / t.ksplit, base = rb / groups, extra = rb - base * groups;
    t.rg = t.wave / t.ksplit;
    t.ks = t.wave - t.rg * t.ksplit;
    t.rb0 = t.rg * base + min(t.rg, extra);
    t.nrb = base + (t.rg < extra ? 1 : 0);
  }
  return true;
}

// The wave's query rows as MFMA operands (rows past the last one are zero).  All rows of the kv head come through LDS once, whole rows by direct loads, each wave
// asking for its share; the chunks of row r lie XOR-permuted by r, so that fragments are read without bank conflicts.  The first key tile is asked for along
// with them where it has room beside them (up to 128 rows), else as soon as they have been read.
template <int D, int WAVES, class FirstTile>
__device__ __forceinline__ void stream_queries(const Ctx &c, const StreamCtx &t, uint4 (&qf)[2][Cfg<true, D>::NF], uint4 *lds, FirstTile first_tile) {
  constexpr int NCH = Cfg<true, D>::NCH, NF = Cfg<true, D>::NF, kRowsPerLoad = 64 / NCH;
  static_assert(256 * NCH <= 2 * KeyTile<true, D>::kChunks, "up to 256 rows in the key tiles' place");
  const Shape &sh = c.sh;
  const uint4 *Q = reinterpret_cast<const uint4 *>(c.Q) + (long long)t.l * sh.qs_layer +
                   (long long)(t.gkv * sh.G) * sh.qs_head + (long long)(t.b * sh.W) * sh.qs_tok;
  const int R = sh.G * sh.W, ln = lane_id_here();
  const bool beside = sh.R_pad * NCH <= KeyTile<true, D>::kChunks;
  for (int r0 = t.wave * kRowsPerLoad; r0 < sh.R_pad; r0 += WAVES * kRowsPerLoad) {
    const int row = r0 + ln / NCH, ch = (ln % NCH) ^ (row & (NCH - 1));
    unsigned r;
    const unsigned head = quotient((unsigned)min(row, R - 1), (unsigned)sh.W, sh.inv_window, r);
    load_to_lds<16>(Q, (head * (unsigned)sh.qs_head + r * (unsigned)sh.qs_tok + (unsigned)ch) * 16u, lds + r0 * NCH);  // (a kv head's rows lie within 4 GiB)
  }
  if (beside) first_tile();
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int row = min(t.rb0 + g, (sh.R_pad >> 5) - 1) * 32 + (ln & 31);
#pragma unroll
    for (int f = 0; f < NF; ++f) qf[g][f] = lds[row * NCH + ((2 * f + (ln >> 5)) ^ (row & (NCH - 1)))];
    if (row >= R) {
#pragma unroll
      for (int f = 0; f < NF; ++f) qf[g][f] = make_uint4(0, 0, 0, 0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();  // the key tiles may overwrite the rows now
  if (!beside) first_tile();
}

// products of the QS row groups of this wave with one block of 32 keys: accumulator rows are keys, lane n owns query row n
template <int D, int QS>
__device__ __forceinline__ void stream_products(f32x16_t (&acc)[QS], const uint4 (&qf)[2][Cfg<true, D>::NF], const char *blk0, const char *blk1) {
  constexpr int NF = Cfg<true, D>::NF;
#pragma unroll
  for (int g = 0; g < QS; ++g)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[g][i] = 0.f;
  // one fragment ahead: the other waves of the SIMD cover the LDS latency, registers are short
  uint4 next = *reinterpret_cast<const uint4 *>(blk0);
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const uint4 kf = next;
    if (f + 1 < NF) next = *reinterpret_cast<const uint4 *>((f & 1 ? blk0 : blk1) + 64 * ((f + 1) >> 1));
#pragma unroll
    for (int g = 0; g < QS; ++g) mma_chunk<true>(acc[g], kf, qf[g][f]);
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(0);
}

// keys that a query row of the window may not see
__device__ __forceinline__ void stream_mask(const Ctx &c, const StreamCtx &t, int rb, int key0, f32x16_t &acc) {
  const int ln = lane_id_here();
  const int limit = row_limit(c.sh, t.s, rb * 32 + (ln & 31)) - key0 - 4 * (ln >> 5);  // row i of the block may be seen up to here
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = acc_row(i, 0) <= limit ? acc[i] : -INFINITY;
}

// First pass.  m: running maximum of a row; zt, zi: its sums of 2^(logit - m) over text and image keys, or (not TRACK) zt over all.
template <int D, int QS, bool TRACK>
__device__ __forceinline__ void stream_stats_block(const Ctx &c, const StreamCtx &t, const uint4 (&qf)[2][Cfg<true, D>::NF], const char *blk0,
                                                   const char *blk1, int key0, unsigned img, float (&m)[2], float (&zt)[2], float (&zi)[2]) {
  constexpr float kLazy = 8.f;  // the running maximum follows once it is 2^8 behind: exact all the same, the sums stay far below overflow
  const float cl = c.sh.scale_log2e;
  f32x16_t acc[QS];
  stream_products<D, QS>(acc, qf, blk0, blk1);
#pragma unroll
  for (int g = 0; g < QS; ++g) {
    if (key0 + 31 > t.s.L - c.sh.W) stream_mask(c, t, t.rb0 + g, key0, acc[g]);
    float tm = fmaxf(acc[g][0], acc[g][1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) tm = fmaxf(fmaxf(tm, acc[g][i]), acc[g][i + 1]);
    tm *= cl;  // cl > 0: the largest logit is the largest product
    if (__any(tm > m[g] + kLazy)) {
      const float M = fmaxf(m[g], tm), f = fast_exp2(m[g] - M);
      zt[g] *= f;
      if constexpr (TRACK) zi[g] *= f;
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
    if constexpr (TRACK) {
      if (img + 1u > 1u) {  // both modalities in this block (rare)
        const unsigned mine = img >> (4 * (lane_id_here() >> 5));
        za = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const bool is_img = (mine >> acc_row(i, 0)) & 1u;
          zi[g] += is_img ? acc[g][i] : 0.f;
          za += is_img ? 0.f : acc[g][i];
        }
      }
      zi[g] += img == 0xffffffffu ? za : 0.f;
      zt[g] += img == 0xffffffffu ? 0.f : za;
    } else {
      zt[g] += za;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// (m, zt, zi) <- fold of two partial statistics of the same row
__device__ __forceinline__ void fold_stats(float &m, float &zt, float &zi, float m2, float zt2, float zi2) {
  const float M = fmaxf(m, m2);  // finite: statistics start at -FLT_MAX
  const float f1 = fast_exp2(m - M), f2 = fast_exp2(m2 - M);
  zt = zt * f1 + zt2 * f2;
  zi = zi * f1 + zi2 * f2;
  m = M;
}

// TRACK: some window of the batch holds image tokens, so a row's mass on text and on image keys is needed apart (the
// second pass sees column sums over rows of both modalities)
template <int D, bool TRACK, int WAVES>
__global__ __launch_bounds__(WAVES * 64, (stream_waves_per_simd<D, WAVES>())) void score_stream_stats_kernel(KernelArgs<Ctx> k) {
  const Ctx &c = k.a;
  using TL = KeyTile<true, D>;
  constexpr int NF = Cfg<true, D>::NF, KT = TL::kRows;
  extern __shared__ uint4 lds[];  // [2] key tiles, then the waves' statistics
  const Shape &sh = c.sh;
  StreamCtx t;
  const ScalarInts meta = first_meta(k, c.meta);
  if (const int own = tiles_grid(sh); (int)blockIdx.x >= own) return place_meta<WAVES * 64>(c, meta, k.meta.n, blockIdx.x - own);
  if (!stream_ctx<D, WAVES>(c, meta, t)) return;
  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)t.l * sh.ks_layer + (long long)t.gkv * sh.ks_head +
                   (long long)t.s.tok_off * sh.ks_tok;
  uint4 qf[2][NF];
  // (tile i of the run in buffer 1 - i % 2: the first one behind the query rows)
  auto buffer = [&](int tile) { return lds + ((tile - t.tile + 1) & 1) * TL::kChunks; };
  stream_queries<D, WAVES>(c, t, qf, lds, [&] { TL::template request<WAVES>(K, sh.ks_tok, t.tile * KT, t.s.L - 1, buffer(t.tile), t.wave); });
  SpanCursor span(meta, t.b);
  // The maxima start finite and below every finite logit: a row whose logits are all -inf keeps sums of 0, no difference of infinities
  float m[2] = {-FLT_MAX, -FLT_MAX}, zt[2] = {0.f, 0.f}, zi[2] = {0.f, 0.f};
  for (int tile = t.tile; tile < t.tile_end; ++tile) {
    __builtin_amdgcn_s_waitcnt(0);  // this wave's part of the tile has landed
    __syncthreads();                // ... and everybody else's; the tile before is no longer read
    if (tile + 1 < t.tile_end)
      TL::template request<WAVES>(K, sh.ks_tok, (tile + 1) * KT, t.s.L - 1, buffer(tile + 1), t.wave);
    const char *base = reinterpret_cast<const char *>(buffer(tile));
    const int ln = lane_id_here();
    const char *rows0 = base + TL::frag_offset(ln & 31, ln >> 5, 0), *rows1 = base + TL::frag_offset(ln & 31, ln >> 5, 1);
#pragma unroll 1
    for (int kb = t.ks; kb < KT / 32; kb += t.ksplit) {
      const int key0 = tile * KT + 32 * kb;
      if (key0 >= t.s.L) break;
      const char *blk0 = rows0 + kb * TL::block_bytes(1), *blk1 = rows1 + kb * TL::block_bytes(1);
      const unsigned img = TRACK ? span.mask(key0, t.s.L) : 0u;
      if (t.nrb == 2) stream_stats_block<D, 2, TRACK>(c, t, qf, blk0, blk1, key0, img, m, zt, zi);
      else stream_stats_block<D, 1, TRACK>(c, t, qf, blk0, blk1, key0, img, m, zt, zi);
    }
  }
  __syncthreads();  // nobody reads keys any more
  float4 *lds_stat = reinterpret_cast<float4 *>(lds);  // [ksplit][R_pad]
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    fold_stats(m[g], zt[g], zi[g], __shfl_xor(m[g], 32, 64), __shfl_xor(zt[g], 32, 64), __shfl_xor(zi[g], 32, 64));
    const int ln = lane_id_here();
    if (g < t.nrb && ln < 32) lds_stat[t.ks * sh.R_pad + (t.rb0 + g) * 32 + ln] = make_float4(m[g], zt[g], zi[g], 0.f);
  }
  __syncthreads();
  float4 *out = c.part_stats + ((long long)(t.l * sh.Hkv + t.gkv) * sh.tiles_score + t.x) * sh.R_pad;
  for (int row = threadIdx.x; row < sh.R_pad; row += WAVES * 64) {
    float4 a = lds_stat[row];
    for (int w = 1; w < t.ksplit; ++w) {
      const float4 o = lds_stat[w * sh.R_pad + row];
      fold_stats(a.x, a.y, a.z, o.x, o.y, o.z);
    }
    out[row] = a;  // (m, sum over text, over image keys), or (m, sum, 0)
  }
}

// Sums over the 32 lanes of each half-wave of sixteen values per lane, halving the values a lane carries at every step
// instead of summing them one by one.  On return lanes with bits b4 b3 b2 hold the sums of v[i + 2 b2 + 4 b3 + 8 b4], i = 0, 1.
__device__ __forceinline__ float2 half_wave_sums(const float (&v)[16]) {
  float w[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    w[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  // The steps inside a row of 16 lanes add with the shifted operand of the other lane group; the second addition of a pair writes
  // only the lane groups whose bit is set (bank_mask).  A value is read by a DPP operand two instructions after it was
  // written at the earliest, which is what the hardware asks for.
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
      : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3])
      : "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]));
  return make_float2(w[0], w[1]);
}

// Second pass.  cr: max + log2(sum) of the rows; part: where the sums over this wave's rows of the block's keys go
template <int D, int QS>
__device__ __forceinline__ void stream_colsum_block(const Ctx &c, const StreamCtx &t, const uint4 (&qf)[2][Cfg<true, D>::NF], const char *blk0,
                                                    const char *blk1, int key0, const float (&cr)[2], float *part) {
  const float cl = c.sh.scale_log2e;
  f32x16_t acc[QS];
  stream_products<D, QS>(acc, qf, blk0, blk1);
  float v[16];
#pragma unroll
  for (int g = 0; g < QS; ++g) {
    if (key0 + 31 > t.s.L - c.sh.W) stream_mask(c, t, t.rb0 + g, key0, acc[g]);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p = fast_exp2(fmaf(acc[g][i], cl, -cr[g]));  // rows past the window: cr = +inf, p = 0
      v[i] = g ? v[i] + p : p;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // (all lanes of a quad have the same sums: they write the same words)
  *reinterpret_cast<float2 *>(part) = half_wave_sums(v);
}

template <int D, bool TRACK, int WAVES>
__global__ __launch_bounds__(WAVES * 64, (stream_waves_per_simd<D, WAVES>())) void score_stream_colsum_kernel(Ctx c) {
  using TL = KeyTile<true, D>;
  constexpr int NF = Cfg<true, D>::NF, KT = TL::kRows;
  extern __shared__ uint4 lds[];  // [2] key tiles
  const Shape &sh = c.sh;
  StreamCtx t;
  const ScalarInts meta = scalar_ints(c.meta);
  if (!stream_ctx<D, WAVES>(c, meta, t)) return;
  float *lds_part = reinterpret_cast<float *>(lds + 2 * TL::kChunks);  // [2][row groups][KT] sums over the rows of a group
  const int row_groups = WAVES / t.ksplit;
  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)t.l * sh.ks_layer + (long long)t.gkv * sh.ks_head +
                   (long long)t.s.tok_off * sh.ks_tok;
  const int R = sh.G * sh.W;
  // The statistics of this wave's rows from all runs of the sequence, folded in the same order by every workgroup (the
  // half-waves take every other run).  The first ones are asked for before the query rows.
  const ScalarInts cu = meta + meta[MW_OFF_CU_SCORE];
  const int x0 = cu[t.b], x1 = cu[t.b + 1];
  const float4 *stats = c.part_stats + (long long)(t.l * sh.Hkv + t.gkv) * sh.tiles_score * sh.R_pad;
  constexpr int kAhead = 4;
  float4 early[2][kAhead];
  {
    const int ln = lane_id_here(), n = ln & 31, half = ln >> 5;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        early[g][u] = stats[(long long)min(x0 + half + 2 * u, x1 - 1) * sh.R_pad + min(t.rb0 + g, (sh.R_pad >> 5) - 1) * 32 + n];
  }
  uint4 qf[2][NF];
  // (tile i of the run in buffer 1 - i % 2: the first one behind the query rows)
  auto buffer = [&](int tile) { return lds + ((tile - t.tile + 1) & 1) * TL::kChunks; };
  stream_queries<D, WAVES>(c, t, qf, lds, [&] { TL::template request<WAVES>(K, sh.ks_tok, t.tile * KT, t.s.L - 1, buffer(t.tile), t.wave); });
  float cr[2], share[2];
  {
    const int ln = lane_id_here(), n = ln & 31, half = ln >> 5;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int row = min(t.rb0 + g, (sh.R_pad >> 5) - 1) * 32 + n;
      float m = -FLT_MAX, zt = 0.f, zi = 0.f;
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (x0 + half + 2 * u < x1) fold_stats(m, zt, zi, early[g][u].x, early[g][u].y, early[g][u].z);
      for (int x = x0 + half + 2 * kAhead; x < x1; x += 2) {
        const float4 o = stats[(long long)x * sh.R_pad + row];
        fold_stats(m, zt, zi, o.x, o.y, o.z);
      }
      fold_stats(m, zt, zi, __shfl_xor(m, 32, 64), __shfl_xor(zt, 32, 64), __shfl_xor(zi, 32, 64));
      const float z = zt + zi;
      // exp2(logit - cr) is the normalised probability
      cr[g] = row < R && z > 0.f ? m + __builtin_amdgcn_logf(z) : INFINITY;
      share[g] = 0.f;
      if (TRACK && t.x == x0 && row < R && half == 0 && z > 0.f) share[g] = (c.mod[t.s.tok_off + t.s.L - sh.W + window_row(sh, row)] ? zt : zi) / z;
    }
  }
  // Cross-modal mass of the kv head's rows.  TRACK: the first run's workgroup adds up the shares of the rows.  Otherwise all rows are text and their mass on image
  // keys is what the importances of those keys add up to (in store_tile).
  float *cross_out = c.cross_part + (long long)(t.l * sh.Hkv + t.gkv) * sh.tiles_score + t.x;
  if constexpr (TRACK) {
    const float v = wave_sum(share[0]) + (t.nrb > 1 ? wave_sum(share[1]) : 0.f);
    if (t.ks == 0 && lane_id_here() == 0) lds_part[t.rg] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      float sum = 0.f;
      for (int i = 0; i < row_groups; ++i) sum += lds_part[i];
      *cross_out = sum;
    }
  }
  float cross = 0.f;
  const float inv_rows = 1.0f / (float)(sh.G * sh.W);
  float *imp = c.importance + (long long)(t.l * sh.Hkv + t.gkv) * sh.T + t.s.tok_off;
  SpanCursor span(meta, t.b);
  auto store_tile = [&](int tile) {  // importances of a finished tile: 64 keys each by the first two waves
    static_assert(KT == 128, "two waves store a tile");
    const int key0 = tile * KT + 64 * t.wave;
    if (t.wave > 1 || key0 >= t.s.L) return;
    const int ln = lane_id_here();
    const float *p = lds_part + (tile & 1) * row_groups * KT + 64 * t.wave + ln;
    float v = 0.f;
    for (int i = 0; i < row_groups; ++i) v += p[i * KT];
    if (key0 + ln < t.s.L) imp[key0 + ln] = v * inv_rows;
    if constexpr (!TRACK) {
      unsigned img = span.mask(key0, t.s.L), img1 = key0 + 32 < t.s.L ? span.mask(key0 + 32, t.s.L) : 0u;
      if (t.s.L - key0 < 64) {  // no keys past the end
        const int left = t.s.L - key0;
        if (left < 32) img &= (1u << left) - 1u;
        else img1 &= (1u << (left - 32)) - 1u;
      }
      cross += ((ln < 32 ? img : img1) >> (ln & 31)) & 1u ? v : 0.f;
    }
  };
  const int ln0 = lane_id_here();
  const int part_lane = (ln0 & 8) + (ln0 & 16) + 4 * (ln0 >> 5) + (ln0 & 4) / 2;  // first of the two keys whose sums this lane ends up with
  for (int tile = t.tile; tile < t.tile_end; ++tile) {
    __builtin_amdgcn_s_waitcnt(0);  // this wave's part of the tile has landed
    __syncthreads();                // ... and everybody else's; the tile before is no longer read, its sums are complete
    if (tile + 1 < t.tile_end)
      TL::template request<WAVES>(K, sh.ks_tok, (tile + 1) * KT, t.s.L - 1, buffer(tile + 1), t.wave);
    if (tile > t.tile) store_tile(tile - 1);
    const char *base = reinterpret_cast<const char *>(buffer(tile));
    const int ln = lane_id_here();
    const char *rows0 = base + TL::frag_offset(ln & 31, ln >> 5, 0), *rows1 = base + TL::frag_offset(ln & 31, ln >> 5, 1);
#pragma unroll 1
    for (int kb = t.ks; kb < KT / 32; kb += t.ksplit) {
      const int key0 = tile * KT + 32 * kb;
      if (key0 >= t.s.L) break;
      const char *blk0 = rows0 + kb * TL::block_bytes(1), *blk1 = rows1 + kb * TL::block_bytes(1);
      float *part = lds_part + ((tile & 1) * row_groups + t.rg) * KT + 32 * kb + part_lane;
      if (t.nrb == 2) stream_colsum_block<D, 2>(c, t, qf, blk0, blk1, key0, cr, part);
      else stream_colsum_block<D, 1>(c, t, qf, blk0, blk1, key0, cr, part);
    }
  }
  __syncthreads();  // the last tile's sums are complete
  store_tile(t.tile_end - 1);
  if constexpr (!TRACK) {
    cross = wave_sum(cross);
    __syncthreads();
    if (threadIdx.x == 64) lds_part[0] = cross;
    __syncthreads();
    if (threadIdx.x == 0) *cross_out = cross + lds_part[0];
  }
}

template <int D, bool TRACK, int WAVES>
hipError_t launch_stream_t(const Ctx &c, const int *words, int n_words) {
  const Shape &sh = c.sh;
  const size_t tiles = 2 * (size_t)KeyTile<true, D>::kChunks * 16;
  const int row_groups = WAVES == 4 ? 1 : sh.R_pad > 128 ? 4 : 2;
  const size_t lds3 = tiles + 2 * (size_t)row_groups * KeyTile<true, D>::kRows * sizeof(float);
  hipError_t e;
  if ((e = allow_full_lds<score_stream_stats_kernel<D, TRACK, WAVES>>()) != hipSuccess) return e;
  if ((e = allow_full_lds<score_stream_colsum_kernel<D, TRACK, WAVES>>()) != hipSuccess) return e;
  if ((long long)sh.n_layers * sh.Hkv * sh.tiles_score + sh.n_spans > 0x7ffffff0LL) return hipErrorInvalidConfiguration;
  const unsigned grid = (unsigned)tiles_grid(sh);
  KernelArgs<Ctx> k;
  fill_kernel_args(k, c, words, n_words);
  {
    ProfScope ps(c.stream, KID_SCORE_STATS);
    score_stream_stats_kernel<D, TRACK, WAVES><<<grid + (n_words ? sh.n_spans : 0), WAVES * 64, tiles, c.stream>>>(k);
  }
  {
    ProfScope ps(c.stream, KID_SCORE_COLSUM);
    score_stream_colsum_kernel<D, TRACK, WAVES><<<grid, WAVES * 64, lds3, c.stream>>>(c);
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_stream(const Ctx &c, const int *words, int n_words) {
  if (stream_waves(c.sh.R_pad) == 4) return c.sh.any_win_img ? launch_stream_t<D, true, 4>(c, words, n_words) : launch_stream_t<D, false, 4>(c, words, n_words);
  return c.sh.any_win_img ? launch_stream_t<D, true, 8>(c, words, n_words) : launch_stream_t<D, false, 8>(c, words, n_words);
}

// ---- the three passes in one kernel, for sequences whose keys fit the registers of one workgroup ----------
// One workgroup per (sequence, kv head, layer), 32*KS keys per wave: K and the query rows come in once instead of
// twice, the row statistics are folded in LDS and two launches go.  Bound by the block loop (see the two kernels above) and, at
// one workgroup per compute unit, by the wait for its keys in front of it: 256 units x 1023 keys x 256 rows
// 74 us (statistics, fold, sums as three kernels) -> 57 us.
template <bool BF16, int D, int WAVES>
__global__ __launch_bounds__(WAVES * 64, (score_waves_per_simd<BF16, D, WAVES>())) void score_resident_kernel(KernelArgs<Ctx> k) {
  const Ctx &c = k.a;
  constexpr int NCH = Cfg<BF16, D>::NCH, NF = Cfg<BF16, D>::NF, KS = score_subs(BF16), THREADS = WAVES * 64;
  extern __shared__ uint4 lds[];
  const Shape &sh = c.sh;
  const ScalarInts meta = first_meta(k, c.meta);
  if ((int)blockIdx.z >= sh.n_layers)
    return place_meta<THREADS>(c, meta, k.meta.n, ((blockIdx.z - sh.n_layers) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
  TileCtx t;
  const UnitBlock ub = unit_block(sh, meta);
  t.b = ub.b; t.gkv = ub.gkv; t.l = ub.l;
  t.s = load_seq(meta, t.b);
  t.wave = threadIdx.x >> 6; t.lane = threadIdx.x & 63; t.n = t.lane & 31; t.half = t.lane >> 5;
  t.key0 = t.wave * 32 * KS;
  t.masked = t.key0 + 32 * KS > t.s.L - sh.W;
  uint4 *ldsq = lds;
  float *lds_stats = reinterpret_cast<float *>(lds + sh.R_pad * (NCH + 1));  // [waves][R_pad]
  RowTables rows;
  rows.c = lds_stats + WAVES * sh.R_pad;
  rows.img = rows.c + sh.R_pad;
  rows.limit = reinterpret_cast<int *>(rows.img + sh.R_pad);
  rows.cross = reinterpret_cast<float *>(rows.limit + sh.R_pad);
  uint4 kf[KS][NF];
  load_keys<BF16, D, KS>(c, t, kf);  // the long way first (HBM); the query rows come from L2
  stage_queries<BF16, D, THREADS>(c, t, ldsq);
  for (int row = t.lane; row < sh.R_pad; row += 64) lds_stats[t.wave * sh.R_pad + row] = -INFINITY;
  fill_row_tables(c, meta, t.b, t.s, rows, WAVES);
  int keymod[KS];
  SpanCursor span(meta, t.b);
#pragma unroll
  for (int sub = 0; sub < KS; ++sub) {
    const int key0 = __builtin_amdgcn_readfirstlane(t.key0) + sub * 32;
    keymod[sub] = key0 < t.s.L ? (span.mask(key0, t.s.L) >> t.n) & 1u : 0;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  const bool mine = t.key0 < t.s.L;  // waves past the end of the sequence have nothing to add
  KeyRegs<BF16, D, KS, WAVES> keys;
#pragma unroll
  for (int sub = 0; sub < KS; ++sub) keys[sub].set(kf[sub]);
  if (mine) {
    if (t.masked) stats_body<BF16, D, KS, WAVES, true>(c, t, keys, ldsq, lds_stats);
    else stats_body<BF16, D, KS, WAVES, false>(c, t, keys, ldsq, lds_stats);
  }
  __syncthreads();
  for (int row = threadIdx.x; row < sh.R_pad; row += THREADS) {
    float m = -INFINITY, z = 0.f;
    if (row < sh.G * sh.W) {
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const float o = lds_stats[w * sh.R_pad + row];
        stat_combine(m, z, o, o == -INFINITY ? 0.f : 1.f);
      }
    }
    rows.c[row] = z > 0.f ? m + __builtin_amdgcn_logf(z) : INFINITY;
  }
  __syncthreads();
  if (mine) {
    float colsum[KS];
#pragma unroll
    for (int sub = 0; sub < KS; ++sub) colsum[sub] = 0.f;
    colsum_any<BF16, D, KS, WAVES>(c, t, keys, keymod, ldsq, rows, colsum);
    store_importance<KS>(c, t, colsum);
  }
  __syncthreads();
  store_cross(c, t, rows, WAVES, t.b);
}

template <bool BF16, int D, int WAVES>
hipError_t launch_resident(const Ctx &c, const int *words, int n_words) {
  const hipError_t e = allow_full_lds<score_resident_kernel<BF16, D, WAVES>>();
  if (e != hipSuccess) return e;
  KernelArgs<Ctx> k;
  fill_kernel_args(k, c, words, n_words);
  const int of_layer = c.sh.batch * c.sh.Hkv, more = n_words ? (c.sh.n_spans + of_layer - 1) / of_layer : 0;  // (a workgroup for every span)
  ProfScope ps(c.stream, KID_SCORE_RESIDENT);
  score_resident_kernel<BF16, D, WAVES><<<dim3(c.sh.batch, c.sh.Hkv, c.sh.n_layers + more), WAVES * 64, score_resident_lds(c.sh, WAVES), c.stream>>>(k);
  return hipGetLastError();
}

template <bool BF16, int D>
hipError_t launch_score_r(const Ctx &c, const int *words, int n_words) {
  if (c.sh.score_resident) return c.sh.score_resident == 8 ? launch_resident<BF16, D, 8>(c, words, n_words) : launch_resident<BF16, D, 16>(c, words, n_words);
  if constexpr (BF16)
    if (c.sh.score_stream) return launch_stream<D>(c, words, n_words);
  return c.sh.score_tpw > 1 ? launch_score_t<BF16, D, true>(c, words, n_words) : launch_score_t<BF16, D, false>(c, words, n_words);
}

}  // namespace

// Waves of the one-workgroup-per-unit kernel, or 0 where the kernels over key tiles do it.
// Times are of the whole plan, us.  Eight waves (up to 512 bf16 keys) beat two kernels except for more than 128 rows of few units, which
// streaming spreads over more workgroups (224 rows x 512 keys: 112 units 49.5, streaming 44.9; 160 units 53.8 and 56.4; 160 rows x 300 keys: 40 units
// 49.8 and 47.9, 112 units 52.3 and 55.1).  Sixteen waves fill a compute unit, so with up to half as many units as compute units (a third, where
// the rows are fewer) the others win: the streaming kernels in bf16 (256 rows x 1000 keys: 32 units 64.5, streaming 41.5; 160 units 77.9 and 79.7;
// 64 rows x 700 keys: 4 units 53.9 and 50.0, 112 units 60.4 and 62.7), the three kernels in fp32 (256 rows x 400 keys: 167 and 112) but for 32 rows of 64
// channels, where a launch is worth more than a second workgroup.  From two units per compute unit on the streaming kernels win again (256 rows x
// 1000 keys, 512 units: 0.95), and where the shorter ones of unequal sequences leave waves idle (128 rows, 512 units x {1000, 200} keys: 186 and 168): three in ten of them, with 32 rows of
// 128 channels six or seven in ten (ten sequences, whole calls, us, resident and streamed: 960 units x {1000, 300} keys 215.7 and 223.6, x 9 of 150 beside one of 1000 142.8 and
// 142.8, 1920 units 257.9 and 251.5), with up to 64 rows of 64 channels and 512 units however many (400 units x {1000, 300} 0.97 of the streamed).
int score_resident_waves(const Shape &sh) {
  const int per_wave = 32 * score_subs(sh.bf16);
  const long long units = (long long)sh.batch * sh.Hkv * sh.n_layers;
  const bool many = units > (sh.score_stream && sh.R_pad <= 192 ? 80 : 128);
  for (int waves = 8; waves <= 16; waves += 8) {
    if (sh.maxL > waves * per_wave) continue;
    if (score_resident_lds(sh, waves) > kLdsBytes) return 0;
    if (waves == 8) return !many && sh.score_stream && sh.R_pad > 128 ? 0 : 8;
    const int least = sh.R_pad <= 64 && sh.d == 64 && units <= 512 ? 0 : sh.R_pad <= 32 && sh.d == 128 ? (units <= 512 ? 40 : 30) : 70;  // per cent of the waves that have keys
    const bool idle = (long long)sh.maxL * sh.batch != sh.T && 100ll * sh.T < (long long)least * sh.batch * waves * per_wave;
    if (many) return sh.score_stream && (idle || (sh.R_pad > 128 && units >= 512)) ? 0 : 16;
    return !sh.bf16 && sh.R_pad <= (sh.d == 64 ? 32 : 0) ? 16 : 0;
  }
  return 0;
}

// bf16, up to 256 query rows: beside the kernels that hold the keys in registers and have the query rows in LDS, 112 units (128 of 160 and 192 rows) x {1100, 16000}
// keys, plan and merge in us: 64 rows of 64 channels 67.1 -> 66.5, 479 -> 447; 160 rows 98.0 -> 92.8, 922 -> 900; 192 rows 102 -> 92.7, 936 -> 914;
// 1024 units x 1600 keys x 32 rows 531 -> 515.
bool score_stream_fits(const Shape &sh) { return sh.bf16 && sh.R_pad <= 256; }

size_t score_lds_limit_bytes(const Shape &sh, long long rows) {
  const int nch = sh.d * (sh.bf16 ? 2 : 4) / 16;
  const long long window = (sh.W + 31) / 32 * 32;
  return (size_t)rows * (nch + 1) * 16 + (size_t)kScoreWaves * rows * sizeof(float) + (size_t)window * 4 + (size_t)kScoreWaves * sh.G * 4;
}

hipError_t launch_score(const Ctx &c, const int *words, int n_words) {
  if (c.sh.bf16) return c.sh.d == 128 ? launch_score_r<true, 128>(c, words, n_words) : launch_score_r<true, 64>(c, words, n_words);
  return c.sh.d == 128 ? launch_score_r<false, 128>(c, words, n_words) : launch_score_r<false, 64>(c, words, n_words);
}

}  // namespace flowmm
