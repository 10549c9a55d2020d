// One decode step of attention over the compacted cache (attention-output equation of the paper's
// Preliminary section, o_t = softmax(q_t K^T / sqrt d) V, with K and V the merged rows that
// flowmm_merge wrote): the operation whose cost the paper's decoding-latency table follows as the
// budget shrinks.  Pure streaming: every merged K and V row is read once.
//
// A workgroup takes `chunk` slots of one (sequence, kv head, layer) for all G query heads of the group
// and leaves the output, or, where a sequence has more slots than that, partials that a second kernel
// folds.  The description of the batch (slot ranges, workgroups per sequence) rides in the kernel
// arguments, so a step is one launch, or two with the fold.
//
// fp32 caches (decode_partial_kernel): lanes that together cover one row (16-byte chunks) form a group; a group walks over its
// rows U at a time (all loads of a trip issued before the first use), computes the G dot products
// of a row with shuffles inside the group, and keeps a running (max, sum, weighted V) per query
// head in the exp2 domain.  The groups of a wave, then the waves, are folded in a fixed order.
// bf16 caches (decode_mfma_kernel): see there.
#include <algorithm>
#include <cfloat>
#include <cstring>

#include "device_common.h"
#include "kernels.h"
#include "profile.h"

namespace flowmm {

namespace {

constexpr int kDecodeTail = 1024;  // four per compute unit (512: 0 to 3 us slower, 2048 to all: 0 to 9)
constexpr int kDThreads = 256;
constexpr int kDWaves = kDThreads / 64;

// (m, z, acc) <- fold of two partial softmax states of the same query head
__device__ __forceinline__ void fold_state(float &m, float &z, float *acc, int n, float m2, float z2, const float *acc2) {
  const float M = fmaxf(m, m2);
  const float Ms = M == -INFINITY ? 0.f : M;
  const float s1 = fast_exp2(m - Ms), s2 = fast_exp2(m2 - Ms);
  z = z * s1 + z2 * s2;
  for (int e = 0; e < n; ++e) acc[e] = acc[e] * s1 + acc2[e] * s2;
  m = M;
}

// The last sequence of the launch, lo .. hi - 1, whose task number from bit SHIFT on is not behind i.
template <int SHIFT>
__device__ __forceinline__ int seq_of(const DecodeArgs &a, int i, int lo, int hi) {
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.cu[mid].task >> SHIFT <= i) lo = mid; else hi = mid;
  }
  return lo;
}

struct DecodeTask {
  int b, x, s0, s1, B;  // sequence of the launch, its task's number among all, the task's slots, the sequence's slots
  int gkv, l;
};

// Workgroups are handed out in the order of the linear index, to the eight XCDs in turn.  The last units' tasks (kDecodeTail of them) go
// from the longest to the shortest over all of these units: compute units that are done early take short ones, and what
// starts last is shortest.  Before, units go one after the other, so that long streams cover the starts of short ones (all tasks from the
// longest to the shortest: 1024 units x {72 .. 487} slots 184 us, 176 so), each one task further on: with eight tasks to a unit one
// sequence would stay on one XCD.
// Tasks of a unit in a row throughout -> this, us: 112 units x {160 .. 982} 57 -> 50 (58 with the fold that parts of 512 need), 224 x {529 ..
// 2856} 332 -> 274, 1024 x 8 x {103 .. 291} 155 -> 119, x {99 .. 506} 276 -> 232, 896 x 5 x {127 .. 551} 146 -> 144.
// ORDERED: all this.  It costs a workgroup two more dependent scalar loads than the plain grid (0.3 us), which calls keep that gain
// nothing from it.
template <bool ORDERED>
__device__ __forceinline__ DecodeTask decode_task(const DecodeArgs &a) {
  DecodeTask t;
  int part;
  if constexpr (!ORDERED) {  // grid (tasks, kv heads, layers)
    t.x = blockIdx.x; t.gkv = blockIdx.y; t.l = blockIdx.z;
    t.b = seq_of<0>(a, t.x, max(0, t.x - (a.tasks - a.n_seqs)), min(a.n_seqs, t.x + 1));  // (every sequence has a task: whole ones need no search)
    part = t.x - a.cu[t.b].task;
  } else {  // grid (kv heads, layers, tasks), read by its linear index
    const unsigned lin = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, units = gridDim.x * gridDim.y;
    const unsigned tasks = (unsigned)a.tasks, first = (unsigned)a.mixed * tasks;
    unsigned unit, i;
    if (lin < first) {
      unsigned turn;
      unit = quotient(lin, tasks, a.inv_tasks, i);
      quotient(unit, tasks, a.inv_tasks, turn);
      i = i + turn < tasks ? i + turn : i + turn - tasks;
    } else {
      i = quotient(lin - first, units - (unsigned)a.mixed, a.inv_last, unit);
      unit += (unsigned)a.mixed;
    }
    unsigned gkv;
    t.l = (int)quotient(unit, gridDim.x, a.inv_heads, gkv);
    t.gkv = (int)gkv;
    if ((int)i < a.full) {
      t.b = seq_of<16>(a, (int)i, 0, a.n_seqs);  // (sequences without a full task share their successor's number)
      part = (int)i - (a.cu[t.b].task >> 16);
    } else {
      const int r = (int)i - a.full;
      t.b = a.rest[r >> 2] >> (8 * (r & 3)) & 255;
      part = (a.cu[t.b + 1].task >> 16) - (a.cu[t.b].task >> 16);
    }
    t.x = (a.cu[t.b].task & 0xffff) + part;
  }
  t.B = a.cu[t.b + 1].slot - a.cu[t.b].slot;
  t.s0 = part * a.chunk;
  t.s1 = min(t.B, t.s0 + a.chunk);
  return t;
}

template <int D, int GP, bool ORDERED>
__global__ __launch_bounds__(kDThreads) void decode_partial_kernel(DecodeArgs a) {
  constexpr bool BF16 = false;
  using CF = Cfg<BF16, D>;
  constexpr int LPR = CF::NCH, RPL = 64 / LPR, EPC = CF::kElemsPerChunk, U = 4;
  constexpr int kGroups = kDWaves * RPL;
  __shared__ float lds_state[kDWaves][GP][D + 2];  // per wave and head: acc[D], m, z

  const DecodeTask task = decode_task<ORDERED>(a);
  const int b = task.b, x = task.x, gkv = task.gkv, l = task.l, B = task.B, s0 = task.s0, s1 = task.s1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, rg = lane / LPR, ch = lane % LPR;
  const int gid = wave * RPL + rg;
  const long long unit = (long long)l * a.Hkv + gkv;
  const uint4 *Kc = reinterpret_cast<const uint4 *>(a.K_c) + (unit * a.SB + a.cu[b].slot) * LPR;
  const uint4 *Vc = reinterpret_cast<const uint4 *>(a.V_c) + (unit * a.SB + a.cu[b].slot) * LPR;

  // this lane's channels of the G queries (heads past G are zero and never written)
  float q[GP][EPC];
#pragma unroll
  for (int g = 0; g < GP; ++g) {
    if (a.g0 + g < a.G) {
      const long long qrow = ((long long)l * a.Hq + gkv * a.G + a.g0 + g) * a.batch + a.b0 + b;
      chunk_to_floats<BF16>(reinterpret_cast<const uint4 *>(a.q)[qrow * LPR + ch], q[g]);
    } else {
#pragma unroll
      for (int e = 0; e < EPC; ++e) q[g][e] = 0.f;
    }
  }
  float m[GP], z[GP], acc[GP][EPC];
#pragma unroll
  for (int g = 0; g < GP; ++g) {
    m[g] = -INFINITY;
    z[g] = 0.f;
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[g][e] = 0.f;
  }

  const float cl = a.scale_log2e;
  for (int r0 = s0 + gid; r0 < s1; r0 += kGroups * U) {
    uint4 kc[U], vc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = min(r0 + u * kGroups, s1 - 1);  // a trip past the end reads the last row again; its weight is 0
      kc[u] = Kc[(long long)r * LPR + ch];
      vc[u] = Vc[(long long)r * LPR + ch];
    }
    // the logits of the U rows for every head, then one rescale of the running state per head and trip
    float fv[U][EPC];
    float sl[GP][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float fk[EPC];
      chunk_to_floats<BF16>(kc[u], fk);
      chunk_to_floats<BF16>(vc[u], fv[u]);
      const bool real = r0 + u * kGroups < s1;
#pragma unroll
      for (int g = 0; g < GP; ++g) {
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) dot = fmaf(fk[e], q[g][e], dot);
        dot = group_sum<LPR>(dot);
        sl[g][u] = real ? dot * cl : -INFINITY;
      }
    }
#pragma unroll
    for (int g = 0; g < GP; ++g) {
      float M = m[g];
#pragma unroll
      for (int u = 0; u < U; ++u) M = fmaxf(M, sl[g][u]);
      const float Ms = M == -INFINITY ? 0.f : M;
      const float sc = fast_exp2(m[g] - Ms);
      z[g] *= sc;
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[g][e] *= sc;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float p = fast_exp2(sl[g][u] - Ms);
        z[g] += p;
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[g][e] = fmaf(p, fv[u][e], acc[g][e]);
      }
      m[g] = M;
    }
  }

  // fold the row groups of the wave (fixed tree), then the waves (in order)
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
    for (int g = 0; g < GP; ++g) {
      const float m2 = __shfl_xor(m[g], o, 64), z2 = __shfl_xor(z[g], o, 64);
      float a2[EPC];
#pragma unroll
      for (int e = 0; e < EPC; ++e) a2[e] = __shfl_xor(acc[g][e], o, 64);
      fold_state(m[g], z[g], acc[g], EPC, m2, z2, a2);
    }
  }
  if (rg == 0) {
#pragma unroll
    for (int g = 0; g < GP; ++g) {
#pragma unroll
      for (int e = 0; e < EPC; ++e) lds_state[wave][g][ch * EPC + e] = acc[g][e];
      if (ch == 0) { lds_state[wave][g][D] = m[g]; lds_state[wave][g][D + 1] = z[g]; }
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < GP * D; idx += kDThreads) {
    const int g = idx / D, ci = idx - g * D;
    if (a.g0 + g >= a.G) continue;
    float mm = lds_state[0][g][D], zz = lds_state[0][g][D + 1], av = lds_state[0][g][ci];
#pragma unroll
    for (int w = 1; w < kDWaves; ++w) fold_state(mm, zz, &av, 1, lds_state[w][g][D], lds_state[w][g][D + 1], &lds_state[w][g][ci]);
    const long long head = (long long)l * a.Hq + gkv * a.G + a.g0 + g;
    if (B <= a.chunk) {  // B >= 1: at least one row has been seen
      reinterpret_cast<float *>(a.out)[(head * a.batch + a.b0 + b) * D + ci] = av / zz;
    } else {
      float *part = a.part + (head * a.tasks + x) * (D + 2);
      part[ci] = av;
      if (ci == 0) { part[D] = mm; part[D + 1] = zz; }
    }
  }
}

// ---- bf16 caches: matrix cores for both products ------------------------------------------------
// What bounds this step is the stream of K and V rows, so the kernel is built around keeping loads in
// flight: every wave works through tiles of 16 rows of its own, with one K and one V buffer in LDS that
// it refills by direct global->LDS loads (whole rows, no registers) as soon as the matrix operands have
// been read out of them.  No barrier until the end.
//   logits  : S[key][head] = K tile x queries (v_mfma 16x16x32); up to 16 heads cost what one costs
//   weights : p = exp2(S - m), kept at fp32 precision for the second product by cutting it into three
//             bf16 terms (8 + 8 + 8 bits of mantissa, the differences are exact; a term that would be 0 is
//             2^-126, far below the rounding of any sum that has a row of weight 1 in it, so that an
//             infinite V stays infinite)
//   output  : O[channel][head] += V^T x p (v_mfma 16x16x16, three times): the accumulator layout of S
//             is the operand layout of p, V comes out of LDS transposed (ds_read_b64_tr_b16), and the
//             rescaling factor of a head lies in the lane that holds the head's column of O
// LDS rows are XOR-swizzled by the row number in 16-byte chunks (the lane asks memory for the chunk that
// belongs where its bytes land), so that neither operand read meets bank conflicts.
constexpr int kMWaves = 8;   // waves of a workgroup, or fewer (decode_waves)
constexpr int kMRows = 16;   // rows of a tile
constexpr int kMHeads = 16;  // query heads of a kv group per launch

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// the 16 rows r0 .. r0+15 (clamped to last) of src into a tile buffer, chunk c of row r at slot c ^ (r % NCH)
template <int NCH>
__device__ __forceinline__ void request_tile(const uint4 *src, int r0, int last, uint4 *tile) {
  const int lane = threadIdx.x & 63;
  constexpr int RPI = 64 / NCH;
#pragma unroll
  for (int j = 0; j < kMRows / RPI; ++j) {
    const int r = j * RPI + lane / NCH, ch = (lane % NCH) ^ (r % NCH);
    load_to_lds<16>(src, ((unsigned)min(r0 + r, last) * NCH + ch) * 16u, tile + j * 64);
  }
}

template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// maximum over the lanes l, l^16, l^32, l^48
__device__ __forceinline__ float quad_max(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float quad_sum(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

template <int D, int WAVES, bool ORDERED>
__global__ __launch_bounds__(WAVES * 64, 4) void decode_mfma_kernel(DecodeArgs a) {
  constexpr int NCH = D / 8, KT = D / 32, DT = D / 16;  // chunks per row, k steps of the logits, channel tiles of the output
  constexpr int kLoads = kMRows * NCH / 64;             // load instructions per tile
  extern __shared__ __align__(16) uint4 lds_tiles[];    // [waves][K, V][16 rows][NCH]; at the end the waves' states
  const DecodeTask task = decode_task<ORDERED>(a);
  const int b = task.b, x = task.x, gkv = task.gkv, l = task.l, B = task.B, s0 = task.s0, s1 = task.s1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, n = lane & 15, q4 = lane >> 4;
  const long long unit = (long long)l * a.Hkv + gkv;
  const uint4 *Kc = reinterpret_cast<const uint4 *>(a.K_c) + (unit * a.SB + a.cu[b].slot) * NCH;
  const uint4 *Vc = reinterpret_cast<const uint4 *>(a.V_c) + (unit * a.SB + a.cu[b].slot) * NCH;
  uint4 *tk = lds_tiles + wave * 2 * kMRows * NCH, *tv = tk + kMRows * NCH;
  const int nh = min(kMHeads, a.G - a.g0);
  const int head0 = l * a.Hq + gkv * a.G + a.g0;  // first query head of this launch

  uint4 qf[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t) qf[t] = make_uint4(0, 0, 0, 0);
  if (n < nh) {
    const uint4 *qrow = reinterpret_cast<const uint4 *>(a.q) + ((long long)(head0 + n) * a.batch + a.b0 + b) * NCH + q4;
#pragma unroll
    for (int t = 0; t < KT; ++t) qf[t] = qrow[4 * t];
  }
  __builtin_amdgcn_s_waitcnt(0);  // the counts below are of tile loads alone

  f32x4_t acc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // of head n; z over this lane's keys only.  The maximum starts finite: rows whose logits are all -inf weigh 0, not NaN
  float m = -FLT_MAX, z = 0.f;
  const float cl = a.scale_log2e;
  const int step = WAVES * kMRows;
  int r0 = s0 + wave * kMRows;
  if (r0 < s1) {
    request_tile<NCH>(Kc, r0, s1 - 1, tk);
    request_tile<NCH>(Vc, r0, s1 - 1, tv);
  }
  for (; r0 < s1; r0 += step) {
    const bool more = r0 + step < s1;
    wait_loads<kLoads>();  // the K tile is there, the V tile may still be on its way
    uint4 kf[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) kf[t] = tk[n * NCH + ((4 * t + q4) ^ (n % NCH))];
    wait_lds();
    if (more) request_tile<NCH>(Kc, r0 + step, s1 - 1, tk);
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      bf16x8_t av, bv;
      __builtin_memcpy(&av, &kf[t], 16);
      __builtin_memcpy(&bv, &qf[t], 16);
      s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, s, 0, 0, 0);  // [key 4 q4 + i][head n]
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = r0 + 4 * q4 + i < s1 ? s[i] * cl : -INFINITY;
    const float mt = quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
    if (__any(mt > m)) {  // some head has a new maximum
      const float M = fmaxf(m, mt), f = fast_exp2(m - M);
      z *= f;
#pragma unroll
      for (int t = 0; t < DT; ++t) acc[t] *= f;
      m = M;
    }
    unsigned hi[4], mid[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = fast_exp2(s[i] - m);
      z += p;
      hi[i] = __float_as_uint(p) & 0xffff0000u;
      const float r1 = fmaxf(p - __uint_as_float(hi[i]), FLT_MIN);
      mid[i] = __float_as_uint(r1) & 0xffff0000u;
      lo[i] = __float_as_uint(fmaxf(r1 - __uint_as_float(mid[i]), FLT_MIN));
    }
    auto pack = [](const unsigned (&v)[4]) {
      uint2 w = make_uint2(__builtin_amdgcn_perm(v[1], v[0], 0x07060302u), __builtin_amdgcn_perm(v[3], v[2], 0x07060302u));
      s16x4_t r;
      __builtin_memcpy(&r, &w, 8);
      return r;
    };
    const s16x4_t ph = pack(hi), pm = pack(mid), pl = pack(lo);
    if (more) wait_loads<kLoads>(); else wait_loads<0>();  // the V tile is there
    s16x4_t vf[DT];
    const int vr = 4 * q4 + (n >> 2);  // this lane's row of the 4 x 16 block that its 16 lanes transpose
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      const char *at = reinterpret_cast<const char *>(tv + vr * NCH + ((2 * t + ((n & 3) >> 1)) ^ (vr % NCH))) + 8 * (n & 1);
      vf[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)at);
    }
    wait_lds();
    if (more) request_tile<NCH>(Vc, r0 + step, s1 - 1, tv);
#pragma unroll
    for (int t = 0; t < DT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[t], ph, acc[t], 0, 0, 0);  // [channel 16 t + 4 q4 + i][head n]
#pragma unroll
    for (int t = 0; t < DT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[t], pm, acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < DT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[t], pl, acc[t], 0, 0, 0);
  }
  z = quad_sum(z);

  // the waves' states, folded in wave order
  __syncthreads();  // nobody reads tiles any more
  float *st = reinterpret_cast<float *>(lds_tiles);  // [waves][nh][D + 4]: O, then m, z
  constexpr int SS = D + 4;
  if (n < nh) {
    float *mine = st + (wave * nh + n) * SS;
#pragma unroll
    for (int t = 0; t < DT; ++t) *reinterpret_cast<float4 *>(mine + 16 * t + 4 * q4) = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
    if (q4 == 0) { mine[D] = m; mine[D + 1] = z; }
  }
  __syncthreads();
  const bool whole = B <= a.chunk;
  for (int idx = threadIdx.x; idx < nh * D; idx += WAVES * 64) {
    const int h = idx / D, ci = idx - h * D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) M = fmaxf(M, st[(w * nh + h) * SS + D]);
    float zz = 0.f, av = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float *o = st + (w * nh + h) * SS;
      const float f = fast_exp2(o[D] - M);  // 0 for a wave that had no tile
      zz = fmaf(o[D + 1], f, zz);
      av = fmaf(o[ci], f, av);
    }
    if (whole) {
      reinterpret_cast<uint16_t *>(a.out)[((long long)(head0 + h) * a.batch + a.b0 + b) * D + ci] = (uint16_t)float_to_bf16_bits(av / zz);
    } else {
      float *part = a.part + ((long long)(head0 + h) * a.tasks + x) * (D + 2);
      part[ci] = av;
      if (ci == 0) { part[D] = M; part[D + 1] = zz; }
    }
  }
}

// out[l][h][b] of the sequences that several workgroups have worked on, from their partial states in slot order
template <bool BF16, int D>
__global__ __launch_bounds__(D) void decode_combine_kernel(DecodeArgs a) {
  const int b = blockIdx.x;
  const int x0 = a.cu[b].task & 0xffff, x1 = a.cu[b + 1].task & 0xffff;
  if (x1 - x0 < 2) return;
  const long long head = (long long)blockIdx.z * a.Hq + blockIdx.y;
  const int ci = threadIdx.x;
  const float *part = a.part + (head * a.tasks + x0) * (D + 2);
  float mm = part[D], zz = part[D + 1], av = part[ci];
  for (int sp = 1; sp < x1 - x0; ++sp) {
    const float *p2 = part + (long long)sp * (D + 2);
    fold_state(mm, zz, &av, 1, p2[D], p2[D + 1], &p2[ci]);
  }
  const float o = av / zz;
  const long long at = (head * a.batch + a.b0 + b) * D + ci;
  if constexpr (BF16) reinterpret_cast<uint16_t *>(a.out)[at] = (uint16_t)float_to_bf16_bits(o);
  else reinterpret_cast<float *>(a.out)[at] = o;
}

template <int D, int GP>
hipError_t launch_partial(const DecodeArgs &a, int n_layers, hipStream_t stream) {
  ProfScope ps(stream, KID_DECODE_PARTIAL);
  if (a.mixed < 0) decode_partial_kernel<D, GP, false><<<dim3(a.tasks, a.Hkv, n_layers), kDThreads, 0, stream>>>(a);
  else decode_partial_kernel<D, GP, true><<<dim3(a.Hkv, n_layers, a.tasks), kDThreads, 0, stream>>>(a);
  return hipGetLastError();
}

template <int D, int WAVES>
hipError_t launch_mfma(const DecodeArgs &a, int n_layers, hipStream_t stream) {
  const int nh = a.G - a.g0 < kMHeads ? a.G - a.g0 : kMHeads;
  size_t lds = (size_t)WAVES * 2 * kMRows * D * 2;
  const size_t states = (size_t)WAVES * nh * (D + 4) * sizeof(float);
  if (states > lds) lds = states;
  const hipError_t e = allow_full_lds<decode_mfma_kernel<D, WAVES, false>, decode_mfma_kernel<D, WAVES, true>>();
  if (e != hipSuccess) return e;
  ProfScope ps(stream, KID_DECODE_PARTIAL);
  if (a.mixed < 0) decode_mfma_kernel<D, WAVES, false><<<dim3(a.tasks, a.Hkv, n_layers), WAVES * 64, lds, stream>>>(a);
  else decode_mfma_kernel<D, WAVES, true><<<dim3(a.Hkv, n_layers, a.tasks), WAVES * 64, lds, stream>>>(a);
  return hipGetLastError();
}

template <bool BF16, int D>
hipError_t launch_decode_t(DecodeArgs a, int n_layers, hipStream_t stream) {
  // query heads of a kv group: sixteen of them, or (fp32) a register-sized batch of up to eight, share one pass over the rows
  for (a.g0 = 0; a.g0 < a.G; a.g0 += BF16 ? kMHeads : 8) {
    const int left = a.G - a.g0;
    hipError_t e;
    if constexpr (BF16) e = a.waves == 2 ? launch_mfma<D, 2>(a, n_layers, stream) : a.waves == 4 ? launch_mfma<D, 4>(a, n_layers, stream) : launch_mfma<D, kMWaves>(a, n_layers, stream);
    else e = left > 4 ? launch_partial<D, 8>(a, n_layers, stream)
           : left > 2 ? launch_partial<D, 4>(a, n_layers, stream)
           : left > 1 ? launch_partial<D, 2>(a, n_layers, stream) : launch_partial<D, 1>(a, n_layers, stream);
    if (e != hipSuccess) return e;
  }
  if (a.tasks > a.n_seqs) {
    ProfScope ps(stream, KID_DECODE_COMBINE);
    decode_combine_kernel<BF16, D><<<dim3(a.n_seqs, a.Hq, n_layers), D, 0, stream>>>(a);
  }
  return hipGetLastError();
}

}  // namespace

// Sequences, their slots together, the longest one's.
struct SlotCounts { int n, sum, longest; };

// A sequence in equal parts.  The number of parts is the one
// whose time is shortest by these measured figures (us; they reproduce the best of 700 sweeps of 4 to 1024 units x 32 to 6000 slots
// within 1 % on average where the sequences are equal; of unequal fp32 ones, whose longest one gives the parts' size, within 3 % in 70 shapes):
//   a trip of a workgroup over its rows takes `alone`, or `each` times the workgroups that share the compute unit;
//   `beside` of them run side by side there (registers, LDS), the next ones follow;
//   sequences of unequal lengths a quarter more on average (fitted to a grid without decode_task's order; with it a factor of 1 chooses as well);
//   parts cost the second launch, 2.5 + 0.37 a part, and their partials, written and read at about 1 TB/s together.
// bf16, 7 heads of 128 channels: 16 units x 830 slots 11.6 whole, 9.5 in four parts; 64 x 1600: 20.7 and 16.3 in three; 112 x 830: 14.5 and
// 15.2 in two; 160 x 3277: 51 and 60 in two.  Up to four trips (512 slots) a second launch is never paid back (410 slots: 7.6 and 8.4 at
// 4 units, 9.6 and 11.6 at 112).
// fp32: 4 units x 410 slots 65 whole, 15.4 in sixteen parts; 112 x 830: 141 and 43 in six; 1024 x 3277: 1315 and 997 in three; with one
// head 256 x 410: 17.1 and 20 in two.
static int decode_parts(const Shape &sh, const SlotCounts &s, bool equal) {
  struct Trip { int rows, beside; float alone, each; };
  static constexpr Trip kF32[2][4] = {{{64, 8, 0.5f, 0.5f}, {64, 7, 0.6f, 0.6f}, {64, 5, 0.8f, 0.8f}, {64, 3, 1.4f, 1.1f}},   // 64 channels; 1, 2, 4, 8 heads
                                      {{32, 7, 1.0f, 1.0f}, {32, 7, 1.1f, 1.0f}, {32, 4, 2.2f, 1.6f}, {32, 3, 7.3f, 2.7f}}};  // 128 channels
  static constexpr Trip kBF16[2] = {{kMWaves * kMRows, 4, 0.55f, 0.55f}, {kMWaves * kMRows, 2, 1.1f, 1.1f}};
  const int wide = sh.d == 128;
  const Trip w = sh.bf16 ? kBF16[wide] : kF32[wide][sh.G > 4 ? 3 : sh.G > 2 ? 2 : sh.G - 1];
  if (sh.bf16 && s.longest <= 4 * w.rows) return 1;
  const int per_pass = sh.bf16 ? kMHeads : 8, passes = (sh.G + per_pass - 1) / per_pass;
  const long long units = (long long)sh.n_layers * sh.Hkv;
  auto round = [&](long long wgs) { return wgs ? (wgs * w.each > w.alone ? wgs * w.each : w.alone) : 0.f; };
  int best = 1;
  float shortest = INFINITY;
  for (int p = 1; p <= kDecodeMaxSplits && (p == 1 || 2 * (s.longest / p) >= w.rows); ++p) {
    const int chunk = (s.longest + p - 1) / p;
    long long tasks = equal ? (long long)p * s.n : (s.sum + chunk - 1) / chunk + s.n / 4;  // of a (layer, kv head)
    if (tasks < s.n) tasks = s.n;
    const long long wgs = (units * tasks + 255) / 256;  // on a compute unit
    const int trips = (chunk + w.rows - 1) / w.rows;
    float t = passes * trips * ((float)(wgs / w.beside) * round(w.beside) + round(wgs % w.beside));
    if (!equal) t *= 1.25f;
    if (p > 1) t += 2.5f + 0.37f * p + 8e-6f * (float)(units * tasks * sh.G) * (float)(sh.d + 2);
    if (t < shortest) { shortest = t; best = p; }
  }
  return best;
}

// Slots per workgroup in a launch of the sequences s (of the call's, which differ from them beyond kDecodeSeqs: what a launch leaves waiting is its own).
//
// bf16 sequences that are nearly equal (the longest no more than a fifth above the average) are cut as equal ones are: nothing is there to fill the
// gaps of the last round (us, whole / cut: 130 units x {5000, 4999} 155 / 128, x {2000, 1990} 64 / 57; 128 units 99 / 97).
// Otherwise a sequence is cut only where the fullest compute unit gets much more than its share, three tenths and eight trips: the tasks go from the longest to
// the shortest (order_tasks), 256 at a time, and a cut costs a second launch and the parts' starts.  Behind units whose tasks go one unit after the other
// a compute unit may be left with two of the longest.  Of 170 measured shapes of 8 to 1024 units and 2 to 60 sequences this takes the shorter of the two
// within 0.5 % on average, 11 % at most, where always whole is 1.8 % and always cut 7 % from it (us, whole / cut: 112 units x 8 of 145 to 982 50 / 57; 192 x {200,
// 400, 4000} 78 / 83; 352 x {204 .. 654, 4100} 259 / 212; 40 x {305, 305, 305, 3050, 3050} 42 / 35; 128 x {516, 516, 516, 5161, 5161} 136 / 149).
// The parts are an eighth of a compute unit's share, of four trips at least and six at most.
static int decode_chunk(const Shape &sh, const int *budgets, const SlotCounts &s) {
  const bool equal = (long long)sh.maxB * sh.batch == sh.SB, near = 5LL * s.longest * s.n <= 6LL * s.sum;
  if (sh.bf16 && !near) {
    constexpr int kTrip = kMWaves * kMRows;
    if (s.longest <= 4 * kTrip) return s.longest;  // (as in decode_parts)
    const long long units = (long long)sh.n_layers * sh.Hkv, last = (kDecodeTail + s.n - 1) / s.n, sorted = units < last ? units : last;
    long long fullest = 2LL * s.longest;
    if ((units - sorted) * s.n < 1024) {
      int len[kDecodeSeqs];
      std::copy(budgets, budgets + s.n, len);
      std::sort(len, len + s.n, [](int x, int y) { return x > y; });
      fullest = 0;
      for (long long i = 0; i < sorted * s.n; i += 256) fullest += len[i / sorted];
    }
    if (10 * 256 * (fullest - 8 * kTrip) <= 13 * sorted * s.sum) return s.longest;
    const long long share = units * s.sum / (8 * 256);
    long long chunk = share < 4 * kTrip ? 4 * kTrip : share < 6 * kTrip ? share : 6 * kTrip;
    if (2LL * s.longest <= 3 * chunk) return s.longest;
    if (chunk * kDecodeMaxSplits < s.longest) chunk = (s.longest + kDecodeMaxSplits - 1) / kDecodeMaxSplits;
    return (int)((chunk + kMRows - 1) / kMRows * kMRows);
  }
  const SlotCounts c = sh.bf16 && !equal ? s : SlotCounts{sh.batch, sh.SB, sh.maxB};
  const int parts = decode_parts(sh, c, sh.bf16 || equal);
  return parts == 1 ? c.longest : ((c.longest + parts - 1) / parts + kMRows - 1) / kMRows * kMRows;
}

// Waves of a bf16 workgroup.  Eight have a tile each only from 128 slots on; where there is more than one workgroup per compute unit
// anyway, fewer waves leave room for more of them (8 / 4 / 2 waves, us: 1024 units, 8 x 41 slots 47.5 / 29.5 / 28.0; 256 x 8 x 54 17.2 / 13.0 /
// 12.5; 224 x 7 x 132 21.2 / 20.0 / 20.5; 120 x 197 5.3 / 5.6 / 7.4; 224 x 5 x 681 42.3 / 43.6 / 43.5).  No workgroup gets more than
// eight trips, so that one long sequence among short ones does not keep the others waiting.
static int decode_waves(const Shape &sh, int chunk) {
  const long long wgs = (long long)sh.n_layers * sh.Hkv * sh.batch;
  const int most = chunk < sh.maxB ? chunk : sh.maxB;
  if (wgs >= 1024 && sh.SB <= 64LL * sh.batch && most <= 8 * 2 * kMRows) return 2;
  return wgs >= 384 && sh.SB <= 256LL * sh.batch && most <= 8 * 4 * kMRows ? 4 : kMWaves;
}

// What decode_task<true> reads of the order.  (Only where the order counts: the smallest calls are bound by host time.)
static void order_tasks(DecodeArgs &a, const int *budgets, int units) {
  int n_rest = 0, rest[kDecodeSeqs];  // slots << 8 | sequence
  a.full = 0;
  for (int i = 0; i < a.n_seqs; ++i) {
    a.cu[i].task |= a.full << 16;
    a.full += budgets[i] / a.chunk;
    if (budgets[i] % a.chunk) rest[n_rest++] = budgets[i] % a.chunk << 8 | i;
  }
  a.cu[a.n_seqs].task |= a.full << 16;
  std::sort(rest, rest + n_rest, [](int x, int y) { return x > y; });
  std::memset(a.rest, 0, sizeof(a.rest));
  for (int i = 0; i < n_rest; ++i) a.rest[i >> 2] |= (rest[i] & 255) << (8 * (i & 3));
  const int last = (kDecodeTail + a.tasks - 1) / a.tasks;
  a.mixed = units > last ? units - last : 0;
  a.inv_tasks = 0xffffffffu / (unsigned)a.tasks;
  a.inv_last = 0xffffffffu / (unsigned)(units > last ? last : units);
  a.inv_heads = 0xffffffffu / (unsigned)a.Hkv;
}

hipError_t launch_decode_attention(const Shape &sh, const int *budgets, DecodeArgs a, hipStream_t stream) {
  a.Hq = sh.Hq; a.Hkv = sh.Hkv; a.G = sh.G; a.SB = sh.SB; a.batch = sh.batch; a.scale_log2e = sh.scale_log2e;
  int slot = 0;
  for (a.b0 = 0; a.b0 < sh.batch; a.b0 += kDecodeSeqs) {
    a.n_seqs = sh.batch - a.b0 < kDecodeSeqs ? sh.batch - a.b0 : kDecodeSeqs;
    const int *len = budgets + a.b0;
    SlotCounts s = {a.n_seqs, 0, 0};
    for (int i = 0; i < a.n_seqs; ++i) {
      a.cu[i].slot = slot + s.sum;
      s.sum += len[i];
      if (len[i] > s.longest) s.longest = len[i];
    }
    a.cu[a.n_seqs].slot = slot += s.sum;
    const int chunk = a.chunk = decode_chunk(sh, len, s);
    a.waves = decode_waves(sh, chunk);
    a.tasks = 0;
    for (int i = 0; i < a.n_seqs; ++i) {
      a.cu[i].task = a.tasks;
      a.tasks += len[i] <= chunk ? 1 : (len[i] + chunk - 1) / chunk;
    }
    a.cu[a.n_seqs].task = a.tasks;
    // Not where every workgroup has a compute unit of its own, nor where the longest is less than a tile above the average, or with up to four
    // workgroups per compute unit less than a trip (plain / ordered, us: 352 units x {69, 70} 8.1 / 8.4, 112 x {300, 400, 200} 15.1 / 15.6, 112 x 7
    // of 73 to 115 12.3 / 12.6; 256 x 8 of 87 to 138 27.0 / 26.0, fp32 112 x {200, 400, 1000, 1100} 126 / 76).
    const int units = sh.Hkv * sh.n_layers;
    const long long wgs = (long long)units * a.tasks, above = wgs <= 1024 ? kMWaves * kMRows : kMRows;
    if (wgs > 256 && (long long)s.longest * s.n - s.sum >= above * s.n) order_tasks(a, len, units);
    else a.mixed = -1;
    const hipError_t e = sh.bf16 ? (sh.d == 128 ? launch_decode_t<true, 128>(a, sh.n_layers, stream) : launch_decode_t<true, 64>(a, sh.n_layers, stream))
                                 : (sh.d == 128 ? launch_decode_t<false, 128>(a, sh.n_layers, stream) : launch_decode_t<false, 64>(a, sh.n_layers, stream));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace flowmm
