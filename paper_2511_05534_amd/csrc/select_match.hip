// Steps "flow", "select", "match" and the grouping of the merge's members in one workgroup per (sequence, kv head, layer), for
// sequences whose contraction (evicted tokens x pivots) is too small to be worth a grid of its own.  The method, the passages
// of the paper and the results are those of select.hip, match.hip and merge.hip's first kernel, bit for bit (the same products, norms and
// order of the candidates, so that a near tie falls alike whichever kernels a batch goes to); what goes is the
// trip of every list through memory (tokens to be matched, eligible pivots, their packed K rows and norms, the assignment),
// two launches, and the idle waves of a 512-token tile that holds 200 tokens.
//
// After the split the lists are in LDS.  A wave takes 32 tokens as MFMA operands in registers; where there are fewer
// groups of tokens than waves several waves share one and split its pivots.  The pivots' rows stream through three LDS tiles by
// direct global->LDS loads, straight from K (the lane asks for its row by the list's entry), and their norms are taken from the
// tile.
// Bound by the chain of phases of one workgroup: 256 units x 1023 tokens back to 819: split, match and groups 38 + 35 + 10 us as
// three kernels, 40 here (phase stamps, with norms that were 1.5 us quicker and not the separate kernels' bit for bit: importances and flow 2.5, top-B 4, lists 2.5,
// tokens and first pivots 4, pivot tiles 18, groups 5).
#include "device_common.h"
#include "flow_core.h"
#include "kernels.h"
#include "merge_csr_core.h"
#include "profile.h"
#include "select_core.h"

namespace flowmm {

namespace {

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kKeysPerThread = 4;
constexpr int kTiles = 3;  // pivot tiles in LDS: one is read, two are on their way
static_assert(kThreads == kCsrThreads, "one workgroup runs all steps");
static_assert(kKeysPerThread * kThreads == kSelectMatchTokens, "a thread keeps four importances");
static_assert(kKeysPerThread * kWaves == 64, "one cell of the class-order scan per lane");

struct TailLds {  // byte offsets into the dynamic LDS block
  int imp, assign, kept, ev, pl_slot, pl_tok, w, tiles, total_bytes;
};

__host__ __device__ inline TailLds tail_lds_layout(int maxL, int maxB, int maxE, int tile_bytes) {
  TailLds m;
  int off = 0;
  auto place = [&](int bytes) { const int at = off; off += (bytes + 15) & ~15; return at; };
  const int bp = (maxB + 31) & ~31;
  m.imp = place(maxL * 4);
  m.assign = place(maxL * 4);
  m.kept = place(maxB * 4);
  m.ev = place(maxE * 2);
  m.pl_slot = place(2 * bp * 2);
  m.pl_tok = place(2 * bp * 2);
  m.w = place(kTiles * 128 * 4);
  m.tiles = place(tile_bytes);
  m.total_bytes = off;
  return m;
}

// words per slot of the counting table: as many waves walk tokens as leave the table in the space of the tiles
__host__ inline int tail_csr_shift(int maxB) {
  int shift = 4;
  while (shift > 0 && (size_t)maxB * (1u << shift) * 4 > 72u * 1024u) --shift;
  return shift;
}

template <bool BF16, int D>
constexpr int tiles_bytes() { return kTiles * KeyTile<BF16, D>::kChunks * 16; }

// LDS reads and writes of the workgroup's waves are over; its direct global->LDS loads may still be on their way
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <bool BF16, int D>
__global__ __launch_bounds__(kThreads, 4) void select_match_kernel(Ctx c, int tile_bytes, int csr_shift) {
  using CF = Cfg<BF16, D>;
  using TL = KeyTile<BF16, D>;
  constexpr int NCH = CF::NCH, NF = CF::NF, TG = 32, ROWS = TL::kRows;
  constexpr int kLoads = ROWS / TL::kGroup / kWaves;  // load instructions of a wave per tile
  extern __shared__ __align__(16) char lds_dyn[];
  __shared__ SmallSelectScratch<kThreads> scratch;
  __shared__ int4 lds_wave[kWaves];
  __shared__ int lds_cell[64], lds_scan[kWaves + 1];
  __shared__ float sh_rho;
  __shared__ int sh_total, sh_dropped;
  const Shape &sh = c.sh;
  const TailLds lay = tail_lds_layout(sh.maxL, sh.maxB, sh.maxE, tile_bytes);
  unsigned *lds_imp = reinterpret_cast<unsigned *>(lds_dyn + lay.imp);        // [L] importance bits
  int *lds_assign = reinterpret_cast<int *>(lds_dyn + lay.assign);            // [L]
  int *lds_kept = reinterpret_cast<int *>(lds_dyn + lay.kept);                // [B]
  uint16_t *lds_ev = reinterpret_cast<uint16_t *>(lds_dyn + lay.ev);          // [L - B] tokens to be matched, in class order
  uint16_t *lds_slot = reinterpret_cast<uint16_t *>(lds_dyn + lay.pl_slot);   // [2][Bp] eligible pivots per class: slots
  uint16_t *lds_tok = reinterpret_cast<uint16_t *>(lds_dyn + lay.pl_tok);     // [2][Bp] their positions
  float *lds_w = reinterpret_cast<float *>(lds_dyn + lay.w);                  // [kTiles][ROWS] 1/norm of a tile's rows
  uint4 *lds_tiles = reinterpret_cast<uint4 *>(lds_dyn + lay.tiles);          // [kTiles] tiles of pivot rows

  const int *meta = c.meta;
  const UnitBlock ub = unit_block(sh, meta);
  const int b = ub.b, gkv = ub.gkv, l = ub.l;
  const SeqInfo s = load_seq(meta, b);
  const long long unit = (long long)l * sh.Hkv + gkv;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  int *assign = c.assign + unit * sh.T + s.tok_off;

  // ---- importances in, and (the last wave) the layer's flow ratio ------------------------------------------
  unsigned keys[kKeysPerThread];
  {
    const unsigned *imp = reinterpret_cast<const unsigned *>(c.importance) + unit * sh.T + s.tok_off;
    const int i0 = threadIdx.x * kKeysPerThread;
#pragma unroll
    for (int j = 0; j < kKeysPerThread; ++j) keys[j] = i0 + j < s.L ? imp[i0 + j] : 0u;
  }
  if (wave == kWaves - 1) {
    const float rho = flow_ratio(c, b, l);
    if (lane == 0) {
      sh_rho = rho;
      sh_dropped = 0;
      if (gkv == 0) {
        c.rho[l * sh.batch + b] = rho;
        c.mode[l * sh.batch + b] = (rho > sh.theta) != (sh.invert_flow != 0) ? 1 : 0;
      }
    }
  }
  {
    const int i0 = threadIdx.x * kKeysPerThread;
    if (i0 < s.L) *reinterpret_cast<uint4 *>(lds_imp + i0) = make_uint4(keys[0], keys[1], keys[2], keys[3]);  // (room for whole chunks)
  }
  // ---- top-B split ------------------------------------------------------------------------------------------
  select_top_b_regs<kThreads, kKeysPerThread, true>(keys, s.L, sh.W, s.B, lds_kept, lds_assign, scratch);
  __syncthreads();
  for (int i = threadIdx.x; i < s.B; i += kThreads) c.kept_idx[unit * sh.SB + s.kept_off + i] = lds_kept[i];
  const bool cross = (sh_rho > sh.theta) != (sh.invert_flow != 0);

  // ---- tokens to be matched, in class order (see select.hip) ---------------------------------------------------
  int n_ev[2];
  {
    const int *order = c.cls_order + s.tok_off;
    const int bound = cross ? s.L : s.n_text;
    int tok[kKeysPerThread];
    unsigned flags = 0;
    unsigned long long bal[kKeysPerThread];
#pragma unroll
    for (int j = 0; j < kKeysPerThread; ++j) {
      const int v = j * kThreads + threadIdx.x;
      tok[j] = v < s.L ? (cross ? v : order[v]) : 0;
    }
#pragma unroll
    for (int j = 0; j < kKeysPerThread; ++j) {
      const int v = j * kThreads + threadIdx.x;
      const bool f = v < s.L && lds_assign[tok[j]] == -2;
      flags |= (unsigned)f << j;
      bal[j] = __ballot(f);
      const unsigned long long bal0 = __ballot(f && v < bound);
      if (lane == 0) lds_cell[j * kWaves + wave] = __popcll(bal[j]) | (__popcll(bal0) << 16);
    }
    __syncthreads();
    const int mine = lds_cell[lane], inc = wave_inclusive_scan(mine);  // every wave scans the cells by itself
    const int total = __builtin_amdgcn_readlane(inc, 63);
    n_ev[0] = total >> 16;
    n_ev[1] = (total & 0xffff) - n_ev[0];
#pragma unroll
    for (int j = 0; j < kKeysPerThread; ++j) {
      const int before = __builtin_amdgcn_readlane(inc - mine, j * kWaves + wave) & 0xffff;
      if ((flags >> j) & 1u) lds_ev[before + __popcll(bal[j] & ((1ull << lane) - 1))] = (uint16_t)tok[j];
    }
  }
  // ---- eligible pivots per token class, padded to whole blocks of 32 with copies of the first ---------------------
  const int Bp = (s.B + 31) & ~31;
  int n_pl[2] = {0, 0};
  for (int s0 = 0; s0 < s.B; s0 += kThreads) {
    const int slot = s0 + threadIdx.x;
    int f0 = 0, f1 = 0, tok = 0;
    if (slot < s.B) {
      tok = lds_kept[slot];
      const bool ok = !(__uint_as_float(lds_imp[tok]) > s.tau);
      const int cls = cross ? 0 : c.mod[s.tok_off + tok];
      f0 = ok && cls == 0;
      f1 = ok && cls == 1;
    }
    int tot;
    const int ex = block_exclusive_scan<kThreads, int>(f0 | (f1 << 16), lds_scan, &tot);
    if (f0 | f1) {
      const int pos = f0 ? n_pl[0] + (ex & 0xffff) : Bp + n_pl[1] + (ex >> 16);
      lds_slot[pos] = (uint16_t)slot;
      lds_tok[pos] = (uint16_t)tok;
    }
    n_pl[0] += tot & 0xffff;
    n_pl[1] += tot >> 16;
  }
  __syncthreads();
#pragma unroll
  for (int cls = 0; cls < 2; ++cls) {
    const int np = (n_pl[cls] + 31) & ~31, e = n_pl[cls] + (int)threadIdx.x;
    if (e < np) {
      lds_slot[cls * Bp + e] = lds_slot[cls * Bp];
      lds_tok[cls * Bp + e] = lds_tok[cls * Bp];
    }
    n_pl[cls] = np;
  }

  // ---- match ------------------------------------------------------------------------------------------------------
  const uint4 *K = reinterpret_cast<const uint4 *>(c.K) + (long long)l * sh.ks_layer + (long long)gkv * sh.ks_head +
                   (long long)s.tok_off * sh.ks_tok;
  int dropped = 0;
#pragma unroll 1
  for (int cls = 0; cls < 2; ++cls) {
    const int cn = cls ? n_ev[1] : n_ev[0], np = cls ? n_pl[1] : n_pl[0], nblk = np >> 5;
    const uint16_t *ev = lds_ev + (cls ? n_ev[0] : 0), *pl_tok = lds_tok + cls * Bp, *pl_slot = lds_slot + cls * Bp;
    if (cn == 0) continue;
    if (np == 0) {  // no eligible pivot
      for (int i = threadIdx.x; i < cn; i += kThreads) {
        lds_assign[ev[i]] = -1;
        ++dropped;
      }
      continue;
    }
    const int groups = (cn + TG - 1) / TG, ntiles = (np + ROWS - 1) / ROWS;
    const int split = groups >= kWaves ? 1 : min(kWaves / groups, nblk);  // waves that share a group of tokens
    const int per_round = kWaves / split, ps = wave % split;
    // this wave's share of the rows of tile t of the list, into buffer t % kTiles (past the end the last rows again: every tile is as many loads)
    auto stage = [&](int t, int buf) {
      const int r0 = t * ROWS, ln = lane_id_here(), j = ln / NCH;
      uint4 *tile = lds_tiles + buf * TL::kChunks;
      static_assert(kLoads * kWaves * TL::kGroup == ROWS, "every wave asks for as many groups");
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        const int g = i * kWaves + wave;
        const unsigned tok = pl_tok[min(r0 + g * TL::kGroup, np - TL::kGroup) + j];
        load_to_lds<16>(K, (tok * (unsigned)sh.ks_tok + (unsigned)((ln % NCH) ^ TL::permute(j))) * 16u, tile + g * TL::kGroupChunks);
      }
    };
#pragma unroll 1
    for (int g0 = 0; g0 < groups; g0 += per_round) {
      __syncthreads();  // the lists are complete, nobody reads tiles any more
      const int wv0 = (g0 + wave / split) * TG;
      const bool active = wave < per_round * split && wv0 < cn;
      uint4 kf[NF];
      const int tok = ev[min(wv0 + n, cn - 1)];
      if (active) {
        const uint4 *row = K + (long long)tok * sh.ks_tok + half;
#pragma unroll
        for (int f = 0; f < NF; ++f) kf[f] = row[2 * f];
      } else {
#pragma unroll
        for (int f = 0; f < NF; ++f) kf[f] = make_uint4(0, 0, 0, 0);
      }
      stage(0, 0);
      if (ntiles > 1) stage(1, 1);
      float shift = 0.f;
#pragma unroll
      for (int f = 0; f < NF; ++f) shift = chunk_sumsq_acc<BF16>(kf[f], shift);
      shift += __shfl_xor(shift, 32, 64);
      shift = sqrtf(shift) * 1.001f;  // >= |<token, pivot>| / |pivot| for every pivot
      RowOperand<NF, BF16 ? kPlain : D == 64 ? kSplitOnce : kSplitEachTime> tokens;  // (fp32 rows of 128 channels are split block by block: registers are short)
      tokens.set(kf);
      unsigned best = 0u;
      int bblk = 0;
      for (int t = 0, buf = 0; t < ntiles; ++t, buf = buf == kTiles - 1 ? 0 : buf + 1) {
        // this wave's part of tile t has landed, the next one's may still be on its way
        if (t + 1 < ntiles) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();  // ... and everybody else's; tile t-1 is no longer read
        if (t + 2 < ntiles) stage(t + 2, buf == 0 ? kTiles - 1 : buf - 1);
        const uint4 *tile = lds_tiles + buf * TL::kChunks;
        const int rows = min(ROWS, np - t * ROWS);
        {  // norms: NCH lanes per row (rows past the list hold its last ones again); lane j of a row's lanes finishes its row of trip j
          constexpr int kTrips = ROWS * NCH / kThreads;
          const int ch = threadIdx.x % NCH;
          float mine = 0.f;
#pragma unroll
          for (int j = 0; j < kTrips; ++j) {
            const int r = j * (kThreads / NCH) + threadIdx.x / NCH, rg = r % TL::kGroup;
            const float ss = group_sum<NCH>(chunk_sumsq<BF16>(tile[(r / TL::kGroup) * TL::kGroupChunks + rg * NCH + (ch ^ TL::permute(rg))]));
            mine = ch == j ? ss : mine;
          }
          if (ch < kTrips) lds_w[buf * ROWS + ch * (kThreads / NCH) + threadIdx.x / NCH] = inverse_norm(mine);
        }
        lds_barrier();
        if (!active) continue;
        const char *rows0 = reinterpret_cast<const char *>(tile) + TL::frag_offset(n, half, 0);
        const char *rows1 = reinterpret_cast<const char *>(tile) + TL::frag_offset(n, half, 1);
        const char *wt = reinterpret_cast<const char *>(lds_w + buf * ROWS) + 16 * half;
        const int blk0 = t * (ROWS / 32), blk1 = blk0 + (rows >> 5);
        // the blocks ps, ps + split, .. of the list
        int blk = blk0 + (ps + split - blk0 % split) % split;
#pragma unroll 1
        for (; blk < blk1; blk += split) {
          const int pb = blk - blk0;
          const char *b0 = rows0 + pb * TL::block_bytes(1), *b1 = rows1 + pb * TL::block_bytes(1);
          f32x16_t prod[1], &acc = prod[0];
          auto frag = [&](int f) { return *reinterpret_cast<const uint4 *>((f & 1 ? b1 : b0) + 64 * (f >> 1)); };
          if constexpr (BF16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
            constexpr int kAhead = 2;
            uint4 next[kAhead];
#pragma unroll
            for (int f = 0; f < kAhead; ++f) next[f] = frag(f);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
              const uint4 cur = next[f % kAhead];
              if (f + kAhead < NF) next[f % kAhead] = frag(f + kAhead);
              mma_chunk<BF16>(acc, cur, tokens.f[f]);  // [pivot][token]
            }
          } else {
            f32_products<false>(prod, &tokens, frag, [&](int, int f) { return (K + (long long)tok * sh.ks_tok + half)[2 * f]; });
          }
          unsigned m = 0u;
#pragma unroll
          for (int g = 0; g < 4; ++g) {  // (see match.hip)
            const float4 w4 = *reinterpret_cast<const float4 *>(wt + pb * 128 + 32 * g);
            const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
              const int i = 4 * g + j;
              const unsigned p0 = (__float_as_uint(fmaf(acc[i], wv[j], shift)) & ~15u) | (unsigned)(15 - i);
              const unsigned p1 = (__float_as_uint(fmaf(acc[i + 1], wv[j + 1], shift)) & ~15u) | (unsigned)(14 - i);
              m = max(max(m, p0), p1);
            }
          }
          if (m > best) { best = m; bblk = blk; }
        }
      }
      if (split > 1) {  // the waves of a group have seen disjoint blocks: the larger candidate wins, the earlier block among equal ones
        __syncthreads();
        uint2 *red = reinterpret_cast<uint2 *>(lds_tiles);  // [waves][64]
        static_assert(kWaves * 64 * sizeof(uint2) <= tiles_bytes<BF16, D>(), "the candidates fit the tiles' space");
        red[wave * 64 + lane] = make_uint2(best, (unsigned)bblk);
        __syncthreads();
        if (ps == 0 && active)
          for (int p = 1; p < split; ++p) {
            const uint2 o = red[(wave + p) * 64 + lane];
            if (o.x > best || (o.x == best && (int)o.y < bblk)) { best = o.x; bblk = (int)o.y; }
          }
      }
      // the two half-waves saw disjoint rows of the same tokens
      int e = bblk * 32 + acc_row(15 - (int)(best & 15u), half);
      const unsigned mine = best >> 4;
      const unsigned other = __shfl_xor(best, 32, 64) >> 4;
      const int oe = __shfl_xor(e, 32, 64);
      if (other > mine || (other == mine && oe < e)) e = oe;
      if (active && ps == 0 && half == 0 && wv0 + n < cn) lds_assign[tok] = pl_slot[e];
    }
  }
  dropped = wave_sum_int(dropped);
  if (lane == 0 && dropped) atomicAdd(&sh_dropped, dropped);
  __syncthreads();
  for (int i = threadIdx.x; i < s.L; i += kThreads) assign[i] = lds_assign[i];
  if (threadIdx.x == 0) c.n_dropped[unit * sh.batch + b] = sh_dropped;
  // ---- members by slot, for the merge that follows in the same call ------------------------------------------------
  if (csr_shift >= 0) merge_csr_body(c, meta, s, b, gkv, l, lds_assign, lds_kept, reinterpret_cast<int *>(lds_tiles), csr_shift, nullptr, lds_wave);
}

template <bool BF16, int D>
int tail_tile_bytes(const Shape &sh) {
  const int table = sh.maxB * 4 << tail_csr_shift(sh.maxB);
  return table > tiles_bytes<BF16, D>() ? table : tiles_bytes<BF16, D>();
}

int tail_tile_bytes(const Shape &sh) {
  if (sh.bf16) return sh.d == 128 ? tail_tile_bytes<true, 128>(sh) : tail_tile_bytes<true, 64>(sh);
  return sh.d == 128 ? tail_tile_bytes<false, 128>(sh) : tail_tile_bytes<false, 64>(sh);
}

template <bool BF16, int D>
hipError_t launch_select_match_t(const Ctx &c, bool with_csr) {
  const Shape &sh = c.sh;
  const hipError_t e = allow_full_lds<select_match_kernel<BF16, D>>();
  if (e != hipSuccess) return e;
  const int tile_bytes = tail_tile_bytes(sh);
  const size_t lds = (size_t)tail_lds_layout(sh.maxL, sh.maxB, sh.maxE, tile_bytes).total_bytes;
  ProfScope ps(c.stream, KID_SELECT_MATCH);
  select_match_kernel<BF16, D><<<dim3(sh.batch, sh.Hkv, sh.n_layers), kThreads, lds, c.stream>>>(c, tile_bytes, with_csr ? tail_csr_shift(sh.maxB) : -1);
  return hipGetLastError();
}

}  // namespace

// One workgroup takes a unit's tokens 512 at a time, each time with a wait for their rows and another walk over the pivots, where the match
// kernel spreads them over workgroups: what counts is how many tokens there are, and with few units (compute units would stand idle)
// their product with the pivots.  One fits a compute unit: from 160 to 256 units, where one round of them fills the chip, twice the tokens pay, and up to
// 512, a second round, they still do with many pivots; with few they cost up to 9 % where that round is half empty, against two to five times the
// scratch.  Time of a call with kernels of their own / with this one (128 channels, inputs that no cache holds):
//   tokens x pivots   16 units  64    112   160   224   256   384   512   1024
//     300 x  600       1.25    1.25  1.28  1.23  1.28  1.29  1.09  1.14  1.12
//    1000 x  200       0.98    1.02  1.09  1.14  1.16  1.14  1.02  1.07  1.04
//    1000 x  600       0.92    0.98  1.09  1.10  1.11  1.16  1.01  1.06  1.01
//    1400 x  200       0.88    0.97  1.01  1.03  1.09  1.09  0.97  1.00  0.97
//    1400 x 1500       0.69    0.76  0.91  0.98  1.10  1.13  0.97  1.06  1.03
//    2000 x  200       0.78    0.89  0.94  1.01  1.03  1.01  0.92  0.95  0.94
//    2000 x  600       0.67    0.82  0.88  0.97  1.02  1.03  0.91  0.97  0.95
// 64 channels: 0.02 less to 0.08 more.  fp32 contractions run at a sixteenth of the rate: 200 x 250 1.10 to 1.16 at 8 to 128 units, 500 x 60 0.98 to 1.13,
// 500 x 120 0.92 to 1.13, 700 x 120 0.74 to 0.99.
bool select_match_fits(const Shape &sh) {
  const long long units = (long long)sh.batch * sh.Hkv * sh.n_layers, candidates = (long long)sh.maxE * sh.maxB;
  if (!sh.rows32 || sh.maxL > kSelectMatchTokens) return false;
  if (sh.bf16 ? sh.maxE > (units >= 160 && units <= 512 ? 2048 : 1024) || (units < 96 && candidates > 300000) : sh.maxE > 512 || candidates > 30000) return false;
  constexpr size_t kStatic = 8 * 1024;
  return (size_t)tail_lds_layout(sh.maxL, sh.maxB, sh.maxE, tail_tile_bytes(sh)).total_bytes <= kLdsBytes - kStatic;
}

hipError_t launch_select_match(const Ctx &c, bool with_csr) {
  if (c.sh.bf16) return c.sh.d == 128 ? launch_select_match_t<true, 128>(c, with_csr) : launch_select_match_t<true, 64>(c, with_csr);
  return c.sh.d == 128 ? launch_select_match_t<false, 128>(c, with_csr) : launch_select_match_t<false, 64>(c, with_csr);
}

}  // namespace flowmm
