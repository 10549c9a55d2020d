// Step "merge": fold every matched non-pivot K/V row into its pivot,
//   out[slot] = (row[pivot] + sum of member rows) / (1 + number of members),
// the uniform-weight instance of the paper's K_merged = f_merge(K, S), V_merged = g_merge(V, S)
// (FlowMM, Preliminary), writing a compacted cache in ascending pivot position.  On request the
// similarity-weighted mean instead (pivot weight 1, member weight max(cosine to the pivot's key, 0),
// computed here from the rows being merged): the variant of the paper's component ablation.
//
// Three kernels, no floating-point atomics, so results are bit-identical from run to run:
//   1. csr   : one workgroup per (sequence, kv head, layer) groups the evicted tokens by slot,
//              ascending inside each slot (a stable counting sort: every wave counts a fixed
//              token range per slot, a scan turns the counts into exact write cursors), and
//              cuts the slots into tasks of at most kTaskChunk members.
//   2. tasks : one wave per task streams its rows with 16-byte loads (a wave covers 64/NCH rows
//              per load), sums them in fp32 and either finishes the slot or leaves a partial.
//   3. fold  : slots with several tasks add up their partials in task order (a few workgroups per
//              (sequence, kv head, layer) walk over them).
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

// Bound by memory: rows gathered at 5.0 to 5.3 TB/s where streaming reaches 5.9.  A wave's chain of round trips is its counts, its task, its
// members, its rows (all of a trip and the next trip's members together).  Whole calls, loads under branches -> this, us: 112 units x
// 4096 tokens in 410 slots 246 -> 227, 256 x 16384 in 819 1862 -> 1844 (this kernel 470 -> 447), in 3277 3241 -> 3096 (610 -> 470).
// WEIGHTED: the similarity-weighted mean (the pivot counts 1, a member max(u, 0), u the cosine of
// its key to the pivot's key, 0 for a zero row; V rows take the weights of their K rows).
template <bool BF16, int D, bool WEIGHTED, bool NEAR>
__global__ __launch_bounds__(256) void merge_tasks_kernel(Ctx c) {
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
    const int4 task = seq_tasks[wl];  // (slot, first member, count, partial index or -1)
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
    if (rg != 0) return;
    if (single) {
      const float den = WEIGHTED ? wsum : (float)(1 + task.z);
#pragma unroll
      for (int e = 0; e < EPC; ++e) { ak[e] = ak[e] / den; av[e] = av[e] / den; }
      K_out[(long long)task.x * LPR + ch] = floats_to_chunk<BF16>(ak);
      V_out[(long long)task.x * LPR + ch] = floats_to_chunk<BF16>(av);
    } else {
      float *p = c.partials + ((unit * sh.part_total + task.w) * 2) * D + ch * EPC;
#pragma unroll
      for (int e = 0; e < EPC; e += 4) {
        *reinterpret_cast<float4 *>(p + e) = make_float4(ak[e], ak[e + 1], ak[e + 2], ak[e + 3]);
        *reinterpret_cast<float4 *>(p + D + e) = make_float4(av[e], av[e + 1], av[e + 2], av[e + 3]);
      }
      if (WEIGHTED && ch == 0) c.partial_w[unit * sh.part_total + task.w] = wsum;
    }
  }
}

// kFoldGroups workgroups per (sequence, kv head, layer) walk over its split slots, one wave per slot.  Bound by the start of the grid and a few dependent
// loads: most split slots have two or three partial sums, so loads past the end stay under their branch (without it, the last one again instead:
// 256 units x 16384 tokens 14.6 -> 16.2 us, 8 ragged prompts 12.8 -> 14.8), and the sequences come in turn (the longest first: 0.4 us more).
template <bool BF16, int D, bool WEIGHTED>
__global__ __launch_bounds__(256) void merge_fold_kernel(Ctx c) {
  constexpr int EPC = Cfg<BF16, D>::kElemsPerChunk;
  constexpr int NCH = Cfg<BF16, D>::NCH;
  const Shape &sh = c.sh;
  const int *meta = c.meta;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int bx = rotated_block_x();
  const int b = bx / kFoldGroups, gkv = blockIdx.y, l = blockIdx.z;
  const long long unit = (long long)l * sh.Hkv + gkv;
  const int n_multi = c.n_multi[unit * sh.batch + b];
  const int q0 = (meta + meta[MW_OFF_CU_MULTI])[b];
  for (int qm = (bx % kFoldGroups) * 4 + wave; qm < n_multi; qm += kFoldGroups * 4) {
    const int q = q0 + qm;
    const SeqInfo s = load_seq(meta, b);
    const int4 e4 = c.multi[unit * sh.multi_total + q];  // (slot, first partial, partials, members)
    const int pivot_tok = c.kept_idx[unit * sh.SB + s.kept_off + e4.x];
    const long long head_off = (long long)l * sh.ks_layer + (long long)gkv * sh.ks_head +
                               (long long)(s.tok_off + pivot_tok) * sh.ks_tok;
    float den = (float)(1 + e4.w);
    if constexpr (WEIGHTED) {
      den = 1.f;  // the pivot's own weight, then the partial sums in task order
      for (int pi = 0; pi < e4.z; ++pi) den += c.partial_w[unit * sh.part_total + e4.y + pi];
    }
    // 2 NCH lanes cover the K and V chunks of the row; the wave's kParts such lane groups share the
    // slot's partials (consecutive ranges, in task order inside each; group 0 starts from the pivot's
    // row) and their sums are added in a fixed tree: the longest chain is 1/kParts of the slot's
    constexpr int kParts = 64 / (2 * NCH);
    {
      const int part_id = lane / (2 * NCH), idx = lane % (2 * NCH);
      const int tensor = idx / NCH, ch = idx % NCH;
      const uint4 *src = reinterpret_cast<const uint4 *>(tensor ? c.V : c.K) + head_off;
      float acc[EPC];
      if (part_id == 0) {
        chunk_to_floats<BF16>(src[ch], acc);
      } else {
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
      }
      const int per = (e4.z + kParts - 1) / kParts;
      const int pbeg = part_id * per, pend = min(e4.z, pbeg + per);
      constexpr int U = 8;  // partials in flight; they are added in task order all the same
      for (int p0 = pbeg; p0 < pend; p0 += U) {
        float part[U][EPC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (p0 + u < pend) {
            const float *pp = c.partials + ((unit * sh.part_total + e4.y + p0 + u) * 2 + tensor) * D + ch * EPC;
#pragma unroll
            for (int e = 0; e < EPC; e += 4) {
              const float4 f4 = *reinterpret_cast<const float4 *>(pp + e);
              part[u][e] = f4.x; part[u][e + 1] = f4.y; part[u][e + 2] = f4.z; part[u][e + 3] = f4.w;
            }
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (p0 + u < pend) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] += part[u][e];
          }
        }
      }
#pragma unroll
      for (int o = 2 * NCH; o < 64; o <<= 1)
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
      if (part_id == 0) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = acc[e] / den;
        const long long orow = (unit * sh.SB + s.kept_off + e4.x) * NCH + ch;
        reinterpret_cast<uint4 *>(tensor ? c.V_out : c.K_out)[orow] = floats_to_chunk<BF16>(acc);
      }
    }
  }
}

template <bool BF16, int D, bool WEIGHTED>
hipError_t launch_merge_w(const Ctx &c) {
  const Shape &sh = c.sh;
  {
    ProfScope ps(c.stream, KID_MERGE_TASKS);
    const dim3 grid((sh.tasks_total + 3) / 4, sh.Hkv, sh.n_layers);
    if (sh.rows32) merge_tasks_kernel<BF16, D, WEIGHTED, true><<<grid, 256, 0, c.stream>>>(c);
    else merge_tasks_kernel<BF16, D, WEIGHTED, false><<<grid, 256, 0, c.stream>>>(c);
  }
  {
    ProfScope ps(c.stream, KID_MERGE_FOLD);
    merge_fold_kernel<BF16, D, WEIGHTED><<<dim3(sh.batch * kFoldGroups, sh.Hkv, sh.n_layers), 256, 0, c.stream>>>(c);
  }
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
