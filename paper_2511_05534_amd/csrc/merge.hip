// Step "merge": fold every matched non-pivot K/V row into its pivot,
//   out[slot] = (row[pivot] + sum of member rows) / (1 + number of members),
// the uniform-weight instance of the paper's K_merged = f_merge(K, S), V_merged = g_merge(V, S)
// (FlowMM, Preliminary), writing a compacted cache in ascending pivot position.  On request the
// similarity-weighted mean instead (pivot weight 1, member weight max(cosine to the pivot's key, 0),
// computed here from the rows being merged): the variant of the paper's component ablation.
//
// Two kernels, no floating-point atomics, so results are bit-identical from run to run:
//   1. csr   : one workgroup per (sequence, kv head, layer) groups the evicted tokens by slot,
//              ascending inside each slot (a stable counting sort: every wave counts a fixed
//              token range per slot, a scan turns the counts into exact write cursors), and
//              cuts the slots into tasks of at most kTaskChunk members.
//   2. tasks : one wave per task streams its rows with 16-byte loads (a wave covers 64/NCH rows
//              per load), sums them in fp32 and either finishes the slot or leaves a partial.  Of a
//              slot with several tasks the wave that ends last adds up the partials in task order.
#include "device_common.h"
#include "kernels.h"
#include "merge_csr_core.h"
#include "profile.h"

namespace flowmm {

namespace {

// Words of LDS in front of the counting table for the pivot positions of the longest budget (a whole number
// of 16-byte chunks), or 0 when table and positions together would not fit: the positions then stay in memory.
__host__ __device__ constexpr int csr_kept_words(int max_budget, int nw_shift) {
  return ((size_t)max_budget << nw_shift) * 4 + (size_t)max_budget * 4 <= 144u * 1024u ? (max_budget + 3) & ~3 : 0;
}

// at most 64 registers: two workgroups of 16 waves then share a compute unit
// members_off: where (in ints from the start of the dynamic LDS) the member list is put together before it
// goes to memory in whole lines, or -1 to write it directly (scattered 4-byte stores: every one of them
// costs a 32-byte memory transaction)
struct CsrArgs {
  Ctx c;
  int nw_shift, members_off;
};
__global__ __launch_bounds__(kCsrThreads, 8) void merge_csr_kernel(KernelArgs<CsrArgs> k) {
  const Ctx &c = k.a.c;
  const int nw_shift = k.a.nw_shift, members_off = k.a.members_off;
  // in front of the counting table the pivot positions of the sequence (the test "is this token its slot's pivot" then
  // needs no second trip to memory behind the token's assignment)
  extern __shared__ int lds_csr[];
  __shared__ int4 lds_wave[kCsrWaves];
  const Shape &sh = c.sh;
  const ScalarInts meta = first_meta(k, c.meta);
  if (blockIdx.x + blockIdx.y + blockIdx.z == 0)  // the words for the kernels behind this one, where it is the call's first
    for (int i = threadIdx.x; i < k.meta.n; i += kCsrThreads) c.meta[i] = meta[i];
  const UnitBlock ub = unit_block(sh, meta);
  const int b = ub.b, gkv = ub.gkv, l = ub.l;
  const SeqInfo s = load_seq(meta, b);
  const long long unit = (long long)l * sh.Hkv + gkv;
  const int *kept = c.kept_idx + unit * sh.SB + s.kept_off;
  const int kept_words = csr_kept_words(sh.maxB, nw_shift);
  if (kept_words)
    for (int i = threadIdx.x; i < s.B; i += kCsrThreads) lds_csr[i] = kept[i];
  merge_csr_body(c, meta, s, b, gkv, l, c.assign + unit * sh.T + s.tok_off, kept_words ? lds_csr : kept, lds_csr + kept_words, nw_shift,
                 members_off >= 0 ? lds_csr + members_off : nullptr, lds_wave);
}

// two floats that a wave of another workgroup may have written in the same launch, or may read in it: past the caches that only one XCD sees
__device__ __forceinline__ void store_shared(float *p, float2 v) {
  unsigned long long u;
  __builtin_memcpy(&u, &v, 8);
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_shared(const float *p) {
  const unsigned long long u = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  float2 v;
  __builtin_memcpy(&v, &u, 8);
  return v;
}

// Bound by memory: rows gathered at 4.8 to 5.3 TB/s (256 units x 16384 tokens, 5 and 50 % kept) where streaming reaches 5.9.  A wave's chain of round trips is its counts, its task, its
// members, its rows (all of a trip and the next trip's members together).  Whole calls, loads under branches -> this, us: 112 units x
// 4096 tokens in 410 slots 246 -> 227, 256 x 16384 in 819 1862 -> 1844 (this kernel 470 -> 447), in 3277 3241 -> 3096 (610 -> 470).
// The partials of a cut-up slot folded by its last wave and not by a kernel of their own, whole calls, us: 112 units x 4096 tokens 220 -> 216, 8 ragged
// prompts 1613 -> 1593, 112 x 900 75.3 -> 72.0, 16 x 3000 tokens of 64 channels 64.1 -> 61.0; 256 x 16384 1833 -> 1832.  Without the bound of 64
// registers (eight waves per SIMD) the ragged prompts lose 4 us where they now gain 20; with it the uniform kernels of bf16 rows keep three to seven registers in scratch, which two partials in flight
// instead of four would free and no call gains by (30 prompts 0.9994).
// WEIGHTED: the similarity-weighted mean (the pivot counts 1, a member max(u, 0), u the cosine of
// its key to the pivot's key, 0 for a zero row; V rows take the weights of their K rows).
template <bool BF16, int D, bool WEIGHTED, bool NEAR>
__global__ __launch_bounds__(256, WEIGHTED ? 4 : 8) void merge_tasks_kernel(Ctx c) {
  using CF = Cfg<BF16, D>;
  constexpr int LPR = CF::NCH;        // lanes that cover one row
  constexpr int RPL = 64 / LPR;       // rows a wave covers per load = row groups of a wave
  constexpr int EPC = CF::kElemsPerChunk;
  constexpr int U = 4;                // loads in flight per lane and tensor
  const Shape &sh = c.sh;
  const int *meta = c.meta;
  const int *cu = meta + meta[MW_OFF_CU_TASK];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // One wave per entry of the task table.  Most slots have a few members or none: RPL such small
  // tasks (whole slot, at most U - 1 members) are done side by side by the row groups of a wave,
  // so the waves at the front of a sequence's range take RPL of them each; the waves at the back of
  // the range stream one larger task each; those in between have nothing to do.
  static_assert(U == kSmallTask, "a small task is the pivot and fewer than U members");
  const int w = blockIdx.x * 4 + wave;
  if (w >= sh.tasks_total) return;
  const int gkv = blockIdx.y, l = blockIdx.z;
  const long long unit = (long long)l * sh.Hkv + gkv;
  const int b = find_seq(cu, meta[MW_BATCH], w);
  const int wl = w - cu[b], room = cu[b + 1] - cu[b];
  const int n_small = c.n_tasks[(unit * sh.batch + b) * 2], n_big = c.n_tasks[(unit * sh.batch + b) * 2 + 1];
  const bool small_wave = wl * RPL < n_small;
  if (!small_wave && wl < room - n_big) return;
  const SeqInfo s = load_seq(meta, b);
  const int rg = lane / LPR, ch = lane % LPR;
  const long long head_off = (long long)l * sh.ks_layer + (long long)gkv * sh.ks_head + (long long)s.tok_off * sh.ks_tok;
  const RowSource<NEAR> K(reinterpret_cast<const uint4 *>(c.K) + head_off, sh.ks_tok, s.L, LPR, ch);
  const RowSource<NEAR> V(reinterpret_cast<const uint4 *>(c.V) + head_off, sh.ks_tok, s.L, LPR, ch);
  const int *kept = c.kept_idx + unit * sh.SB + s.kept_off;
  const int *seq_members = c.members + unit * sh.T + s.tok_off;
  uint4 *K_out = reinterpret_cast<uint4 *>(c.K_out) + (unit * sh.SB + s.kept_off) * LPR;
  uint4 *V_out = reinterpret_cast<uint4 *>(c.V_out) + (unit * sh.SB + s.kept_off) * LPR;
  const int4 *seq_tasks = c.tasks + unit * sh.tasks_total + cu[b];
  // weighted merge: the weight of a member row against the pivot's (the lanes of a row group call together)
  auto weight = [&](const float (&fk)[EPC], const float (&pk)[EPC], float pss) {
    float dot = 0.f, ss = 0.f;
#pragma unroll
    for (int e = 0; e < EPC; ++e) { dot = fmaf(fk[e], pk[e], dot); ss = fmaf(fk[e], fk[e], ss); }
#pragma unroll
    for (int o = LPR / 2; o >= 1; o >>= 1) { dot += __shfl_xor(dot, o, 64); ss += __shfl_xor(ss, o, 64); }
    return ss > 0.f && pss > 0.f ? fmaxf(dot / (sqrtf(ss) * sqrtf(pss)), 0.f) : 0.f;
  };

  // ---- small tasks: the pivot's row and up to U - 1 member rows, summed in that order by one row group
  if (small_wave) {
    if (wl * RPL + rg >= n_small) return;
    const int4 mine = seq_tasks[wl * RPL + rg];  // (slot, first member, count, -1)
    int tokv[U];
    tokv[0] = kept[mine.x];
#pragma unroll
    for (int u = 1; u < U; ++u) tokv[u] = seq_members[mine.y + min(u, max(mine.z, 1)) - 1];  // (past the slot's members: not used)
    uint4 kc[U], vc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      kc[u] = K.row(tokv[u], u <= mine.z);
      vc[u] = V.row(tokv[u], u <= mine.z);
    }
    __builtin_amdgcn_sched_barrier(0);
    float ak[EPC], av[EPC];
    chunk_to_floats<BF16>(kc[0], ak);
    chunk_to_floats<BF16>(vc[0], av);
    float den = (float)(1 + mine.z);
    if constexpr (WEIGHTED) {
      float pk[EPC], pss = 0.f;
#pragma unroll
      for (int e = 0; e < EPC; ++e) { pk[e] = ak[e]; pss = fmaf(pk[e], pk[e], pss); }
#pragma unroll
      for (int o = LPR / 2; o >= 1; o >>= 1) pss += __shfl_xor(pss, o, 64);
      den = 1.f;
#pragma unroll
      for (int u = 1; u < U; ++u) {
        float fk[EPC], fv[EPC];
        chunk_to_floats<BF16>(kc[u], fk);
        chunk_to_floats<BF16>(vc[u], fv);
        const float w = weight(fk, pk, pss);
        den += w;
#pragma unroll
        for (int e = 0; e < EPC; ++e) { ak[e] = fmaf(w, fk[e], ak[e]); av[e] = fmaf(w, fv[e], av[e]); }
      }
    } else {
#pragma unroll
      for (int u = 1; u < U; ++u) {
        if (u <= mine.z) {
          float fk[EPC], fv[EPC];
          chunk_to_floats<BF16>(kc[u], fk);
          chunk_to_floats<BF16>(vc[u], fv);
#pragma unroll
          for (int e = 0; e < EPC; ++e) { ak[e] += fk[e]; av[e] += fv[e]; }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < EPC; ++e) { ak[e] = ak[e] / den; av[e] = av[e] / den; }
    K_out[(long long)mine.x * LPR + ch] = floats_to_chunk<BF16>(ak);
    V_out[(long long)mine.x * LPR + ch] = floats_to_chunk<BF16>(av);
    return;
  }

  // ---- a larger task: all row groups of the wave stream its rows
  {
    int4 task = seq_tasks[wl];  // (slot, first member, count and split slot, partial index or -1)
    const int split_slot = (int)((unsigned)task.z >> kTaskCountBits);
    task.z &= (1 << kTaskCountBits) - 1;
    const int *members = seq_members + task.y;
    const bool single = task.w < 0;
    const int pivot_tok = kept[task.x];
    const auto member = [&](int j) {  // (the last one again past the end)
      return *reinterpret_cast<const int *>(reinterpret_cast<const char *>(members) + 4u * (unsigned)min(j, task.z - 1));
    };
    int tokv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) tokv[u] = member(rg + u * RPL);
    // the pivot's row: the first row group of a whole slot starts from it, and the weighted merge compares with it
    uint4 pk_chunk = K.row(pivot_tok, WEIGHTED || (single && rg == 0)), pv_chunk = V.row(pivot_tok, single && rg == 0);
    uint4 kc[U], vc[U];
    // a trip's rows and the next trip's members: everything is asked for before the first of it is waited for
    auto request = [&](int j0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool real = j0 + rg + u * RPL < task.z;
        kc[u] = K.row(tokv[u], real);
        vc[u] = V.row(tokv[u], real);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) tokv[u] = member(j0 + RPL * U + rg + u * RPL);
      __builtin_amdgcn_sched_barrier(0);
    };
    float ak[EPC], av[EPC];
    float wsum = 0.f;        // weighted merge: weights this row group has added
    float pk[EPC], pss = 0.f;  // weighted merge: this lane's chunk of the pivot's key, its squared norm
    for (int j0 = 0; j0 < task.z; j0 += RPL * U) {
      request(j0);
      if (j0 == 0) {
        // (opaque: hoisted in front of the requests above, the conversion would wait for the pivot's row there)
        asm volatile("" : "+v"(pk_chunk.x), "+v"(pk_chunk.y), "+v"(pk_chunk.z), "+v"(pk_chunk.w), "+v"(pv_chunk.x), "+v"(pv_chunk.y), "+v"(pv_chunk.z), "+v"(pv_chunk.w));
        chunk_to_floats<BF16>(pk_chunk, ak);
        chunk_to_floats<BF16>(pv_chunk, av);
        if constexpr (WEIGHTED) {
          const bool mine = single && rg == 0;
#pragma unroll
          for (int e = 0; e < EPC; ++e) {
            pk[e] = ak[e];
            pss = fmaf(pk[e], pk[e], pss);
            ak[e] = mine ? ak[e] : 0.f;
          }
          wsum = mine ? 1.f : 0.f;
#pragma unroll
          for (int o = LPR / 2; o >= 1; o >>= 1) pss += __shfl_xor(pss, o, 64);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {  // rows past the end are zeros
        float fk[EPC], fv[EPC];
        chunk_to_floats<BF16>(kc[u], fk);
        chunk_to_floats<BF16>(vc[u], fv);
        if constexpr (WEIGHTED) {
          const float w = weight(fk, pk, pss);
          wsum += w;
#pragma unroll
          for (int e = 0; e < EPC; ++e) { ak[e] = fmaf(w, fk[e], ak[e]); av[e] = fmaf(w, fv[e], av[e]); }
        } else {
#pragma unroll
          for (int e = 0; e < EPC; ++e) { ak[e] += fk[e]; av[e] += fv[e]; }
        }
      }
    }
    // fold the row groups (fixed tree)
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        ak[e] += __shfl_xor(ak[e], o, 64);
        av[e] += __shfl_xor(av[e], o, 64);
      }
      if constexpr (WEIGHTED) wsum += __shfl_xor(wsum, o, 64);
    }
    if (single) {
      if (rg != 0) return;
      const float den = WEIGHTED ? wsum : (float)(1 + task.z);
#pragma unroll
      for (int e = 0; e < EPC; ++e) { ak[e] = ak[e] / den; av[e] = av[e] / den; }
      K_out[(long long)task.x * LPR + ch] = floats_to_chunk<BF16>(ak);
      V_out[(long long)task.x * LPR + ch] = floats_to_chunk<BF16>(av);
      return;
    }
    // A part of a slot: its sums go past the caches to where every XCD sees them, and once they are there the wave adds itself to the parts that are. The one that
    // finds the others there (none waits) folds them all, in task order whoever it is.
    float *part = c.partials + (unit * sh.part_total + task.w) * 2 * D + ch * EPC;
    if (rg == 0) {
#pragma unroll
      for (int e = 0; e < EPC; e += 2) {
        store_shared(part + e, make_float2(ak[e], ak[e + 1]));
        store_shared(part + D + e, make_float2(av[e], av[e + 1]));
      }
      if (WEIGHTED && ch == 0) __hip_atomic_store(c.partial_w + unit * sh.part_total + task.w, wsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    int4 *slot = c.multi + unit * sh.multi_total + (meta + meta[MW_OFF_CU_MULTI])[b] + split_slot;
    const int n_members = slot->x, first = slot->y, n_parts = slot->z;
    // Arrived.  By the memory model nothing orders the relaxed stores above before the count, or the count before the relaxed loads below.  What does is
    // this chip: a store of agent scope is acknowledged when it is where the loads of that scope look, and the wave counts itself once all of its stores have
    // been (neither they nor the count can cross the wait: it clobbers memory).  (A release of agent scope would write the L2's other lines back too, every
    // time: 256 units x 16384 tokens 1804 -> 2310 us.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int there = 0;
    if (lane == 0) there = __hip_atomic_fetch_add(&slot->w, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(there) != n_parts - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    float den = (float)(1 + n_members);
    if constexpr (WEIGHTED) {
      den = 1.f;  // the pivot's own weight, then the partial sums in task order
      for (int p = 0; p < n_parts; ++p) den += __hip_atomic_load(c.partial_w + unit * sh.part_total + first + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // 2 LPR lanes cover the K and V chunks of the row; the wave's kParts such lane groups share the
    // slot's partials (consecutive ranges, in task order inside each; group 0 starts from the pivot's
    // row) and their sums are added in a fixed tree: the longest chain is 1/kParts of the slot's
    constexpr int kParts = 64 / (2 * LPR);
    const int part_id = lane / (2 * LPR), tensor = lane / LPR % 2;
    float acc[EPC];
    const uint4 k_row = K.row(pivot_tok, part_id == 0 && tensor == 0), v_row = V.row(pivot_tok, part_id == 0 && tensor == 1);  // (zeros in the other groups)
    chunk_to_floats<BF16>(tensor ? v_row : k_row, acc);
    const int per = (n_parts + kParts - 1) / kParts;
    const int pbeg = part_id * per, pend = min(n_parts, pbeg + per);
    constexpr int UF = 4;  // partials in flight; they are added in task order all the same
    for (int p0 = pbeg; p0 < pend; p0 += UF) {
      float2 v[UF][EPC / 2];
#pragma unroll
      for (int u = 0; u < UF; ++u)
        if (p0 + u < pend) {
          const float *pp = c.partials + ((unit * sh.part_total + first + p0 + u) * 2 + tensor) * D + ch * EPC;
#pragma unroll
          for (int e = 0; e < EPC; e += 2) v[u][e / 2] = load_shared(pp + e);
        }
#pragma unroll
      for (int u = 0; u < UF; ++u)
        if (p0 + u < pend) {
#pragma unroll
          for (int e = 0; e < EPC; e += 2) { acc[e] += v[u][e / 2].x; acc[e + 1] += v[u][e / 2].y; }
        }
    }
#pragma unroll
    for (int o = 2 * LPR; o < 64; o <<= 1)
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
    if (part_id != 0) return;
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = acc[e] / den;
    (tensor ? V_out : K_out)[(long long)task.x * LPR + ch] = floats_to_chunk<BF16>(acc);
  }
}

template <bool BF16, int D, bool WEIGHTED>
hipError_t launch_merge_w(const Ctx &c) {
  const Shape &sh = c.sh;
  ProfScope ps(c.stream, KID_MERGE_TASKS);
  const dim3 grid((sh.tasks_total + 3) / 4, sh.Hkv, sh.n_layers);
  if (sh.rows32) merge_tasks_kernel<BF16, D, WEIGHTED, true><<<grid, 256, 0, c.stream>>>(c);
  else merge_tasks_kernel<BF16, D, WEIGHTED, false><<<grid, 256, 0, c.stream>>>(c);
  return hipGetLastError();
}

template <bool BF16, int D>
hipError_t launch_merge_t(const Ctx &c) {
  return c.sh.weighted_merge ? launch_merge_w<BF16, D, true>(c) : launch_merge_w<BF16, D, false>(c);
}

}  // namespace

// largest per-sequence budget decides how many waves may walk tokens: the [B][NW] table lives in LDS
static int merge_csr_wave_shift(int max_budget) {
  int shift = 4;  // 16 waves
  while (shift > 0 && (size_t)max_budget * (1u << shift) * 4 > 128u * 1024u) --shift;
  return shift;
}

size_t merge_csr_lds_bytes(int max_budget) {
  const int shift = merge_csr_wave_shift(max_budget);
  return (((size_t)max_budget << shift) + csr_kept_words(max_budget, shift)) * 4;
}

hipError_t launch_merge_csr(const Ctx &c, const int *words, int n_words) {
  const Shape &sh = c.sh;
  const size_t lds = merge_csr_lds_bytes(sh.maxB);
  hipError_t e = allow_full_lds<merge_csr_kernel>();
  if (e != hipSuccess) return e;
  // the member list is put together in LDS when that leaves the compute units as many workgroups as before:
  // two each, or one each when there are no more workgroups than compute units
  const size_t with_members = lds + (size_t)sh.maxE * 4;
  const long long wgs = (long long)sh.batch * sh.Hkv * sh.n_layers;
  // (short lists are not worth the extra pass over them: 19 against 23 us at 3700 members per list)
  const bool stage = sh.maxE >= 8192 &&
                     (with_members <= kLdsBytes / 2 - 1024 || (wgs <= 256 && with_members <= kLdsBytes - 8 * 1024));
  ProfScope ps(c.stream, KID_MERGE_CSR);
  KernelArgs<CsrArgs> k;
  fill_kernel_args(k, CsrArgs{c, merge_csr_wave_shift(sh.maxB), stage ? (int)(lds / 4) : -1}, words, n_words);
  merge_csr_kernel<<<dim3(sh.batch, sh.Hkv, sh.n_layers), kCsrThreads, stage ? with_members : lds, c.stream>>>(k);
  return hipGetLastError();
}

hipError_t launch_merge(const Ctx &c, bool with_csr, const int *words, int n_words) {
  const hipError_t e = with_csr ? launch_merge_csr(c, words, n_words) : hipSuccess;
  if (e != hipSuccess) return e;
  if (c.sh.bf16) return c.sh.d == 128 ? launch_merge_t<true, 128>(c) : launch_merge_t<true, 64>(c);
  return c.sh.d == 128 ? launch_merge_t<false, 128>(c) : launch_merge_t<false, 64>(c);
}

}  // namespace flowmm
