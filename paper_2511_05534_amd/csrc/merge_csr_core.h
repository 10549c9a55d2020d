// Grouping of the evicted tokens of one (sequence, kv head, layer) by slot, shared by the stand-alone CSR kernel (merge.hip) and the
// kernel that splits, matches and groups short sequences in one workgroup (select_match.hip).
#pragma once
#include "device_common.h"
#include "kernels.h"
#include "select_core.h"

namespace flowmm {

constexpr int kCsrThreads = kCsrWaves * 64;
constexpr int kCsrAhead = 4;   // rounds of 64 tokens a walking wave loads ahead
constexpr int kSmallTask = 4;  // a slot with fewer members is merged by one row group (pivot + members = loads in flight)

// Exclusive scan over the workgroup of four counters at once; *total gets the sums over all threads.  The lanes scan by DPP operands
// and every wave adds up the totals of the waves before it by itself, so a scan is two barriers.
__device__ __forceinline__ int4 block_exclusive_scan4(int4 v, int4 *lds_wave, int4 *total) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int4 inc = make_int4(wave_inclusive_scan(v.x), wave_inclusive_scan(v.y), wave_inclusive_scan(v.z), wave_inclusive_scan(v.w));
  __syncthreads();
  if (lane == 63) lds_wave[wave] = inc;
  __syncthreads();
  const int4 w = lane < kCsrWaves ? lds_wave[lane] : make_int4(0, 0, 0, 0);
  const int4 winc = make_int4(wave_inclusive_scan(w.x), wave_inclusive_scan(w.y), wave_inclusive_scan(w.z), wave_inclusive_scan(w.w));
  auto at = [](int x, int l) { return __builtin_amdgcn_readlane(x, l); };
  *total = make_int4(at(winc.x, 63), at(winc.y, 63), at(winc.z, 63), at(winc.w, 63));
  return make_int4(at(winc.x - w.x, wave) + inc.x - v.x, at(winc.y - w.y, wave) + inc.y - v.y, at(winc.z - w.z, wave) + inc.z - v.z,
                   at(winc.w - w.w, wave) + inc.w - v.w);
}

// How many lower lanes of the wave hold the same slot as this lane, and how many lanes do in all (only
// meaningful where member).  One ballot per slot bit; the lanes that agree with this one on the bit
// are ballot XNOR (bit ? ~0 : 0), taken on the two halves of the wave mask.
__device__ __forceinline__ void same_slot_rank(bool member, int slot, int nbits, int &below, int &total) {
  const unsigned long long mm = __ballot(member);
  unsigned lo = (unsigned)mm, hi = (unsigned)(mm >> 32);
  for (int bit = 0; bit < nbits; ++bit) {
    const unsigned e = 0u - ((unsigned)(slot >> bit) & 1u);  // all ones where the bit is set
    const unsigned long long bb = __ballot(member && e != 0u);
    lo &= ~((unsigned)bb ^ e);
    hi &= ~((unsigned)(bb >> 32) ^ e);
  }
  below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
  total = __popc(lo) + __popc(hi);
}

// All kCsrThreads threads call.  assign [L] and kept [B]: the sequence's, in LDS or memory; lds_tbl: [1 << nw_shift][B] words of LDS, cleared
// here: per-wave counts, later write cursors (the slot runs fastest, so that the slots of a wave's 64 tokens and the 1024 slots
// of a scan step fall on different banks); lds_members: [evicted tokens] words of LDS in which the member list is put together
// before it goes to memory in whole lines, or null.
template <class Ints>
__device__ __forceinline__ void merge_csr_body(const Ctx &c, Ints meta, const SeqInfo &s, int b, int gkv, int l, const int *assign, const int *kept,
                                               int *lds_tbl, int nw_shift, int *lds_members, int4 *lds_wave) {
  const Shape &sh = c.sh;
  const long long unit = (long long)l * sh.Hkv + gkv;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int NW = 1 << nw_shift;  // waves that walk tokens (the table must fit in LDS)
  int *members = c.members + unit * sh.T + s.tok_off;
  int *seg_off = c.seg_off + unit * (sh.SB + sh.batch) + s.kept_off + b;
  const int task_base = (meta + meta[MW_OFF_CU_TASK])[b];
  const int task_room = (meta + meta[MW_OFF_CU_TASK])[b + 1] - task_base;
  const int multi_base = (meta + meta[MW_OFF_CU_MULTI])[b];
  const int part_base = (meta + meta[MW_OFF_CU_PART])[b];
  int4 *tasks = c.tasks + unit * sh.tasks_total + task_base;
  int4 *multi = c.multi + unit * sh.multi_total + multi_base;

  int nbits = 0;
  while ((1 << nbits) < s.B) ++nbits;
  const int range = ((s.L + NW - 1) / NW + 63) & ~63;  // tokens per walking wave
  const int r0 = wave * range, r1 = min(s.L, r0 + range);

  for (int i = threadIdx.x; i < s.B * NW; i += kCsrThreads) lds_tbl[i] = 0;
  __syncthreads();

  // pass 1: members of each slot inside each wave's token range (kCsrAhead rounds of 64 tokens have
  // their two dependent loads in flight together)
  if (wave < NW) {
    for (int i0 = r0; i0 < r1; i0 += 64 * kCsrAhead) {
      int slotv[kCsrAhead], keptv[kCsrAhead];
#pragma unroll
      for (int u = 0; u < kCsrAhead; ++u) {
        const int i = i0 + 64 * u + lane;
        slotv[u] = i < r1 ? assign[i] : -1;
      }
#pragma unroll
      for (int u = 0; u < kCsrAhead; ++u) keptv[u] = slotv[u] >= 0 ? kept[slotv[u]] : -1;
#pragma unroll
      for (int u = 0; u < kCsrAhead; ++u) {
        if (i0 + 64 * u >= r1) break;
        const int i = i0 + 64 * u + lane, slot = slotv[u];
        // counting needs no order: the few lanes of a round that share a slot take their turns in the LDS
        if (slot >= 0 && keptv[u] != i) atomicAdd(&lds_tbl[wave * s.B + slot], 1);
      }
    }
  }
  __syncthreads();

  // scan over slots: segment offsets, write cursors, task list
  // A slot with fewer than kSmallTask members is a small task (a row group of the task kernel does it
  // alone); the small tasks fill the sequence's range of the table from the front, the others from the back.
  int seg_carry = 0, small_carry = 0, task_carry = 0, multi_carry = 0, part_carry = 0;
  for (int s0 = 0; s0 < s.B; s0 += kCsrThreads) {
    const int slot = s0 + threadIdx.x;
    int n = 0;
    if (slot < s.B)
      for (int w = 0; w < NW; ++w) n += lds_tbl[w * s.B + slot];
    const int nt = slot < s.B ? max(1, (n + kTaskChunk - 1) / kTaskChunk) : 0;
    const int is_multi = nt > 1;
    const int is_small = slot < s.B && n < kSmallTask;
    int4 tot;  // members, small tasks and (upper half) split slots, other tasks, partials
    const int4 ex = block_exclusive_scan4(make_int4(n, is_small | (is_multi << 16), is_small ? 0 : nt, is_multi ? nt : 0), lds_wave, &tot);
    const int seg = seg_carry + ex.x, sb = small_carry + (ex.y & 0xffff), mb = multi_carry + (ex.y >> 16);
    const int tb = task_carry + ex.z, pb = part_carry + ex.w;
    const int tot_n = tot.x, tot_s = tot.y & 0xffff, tot_m = tot.y >> 16, tot_t = tot.z, tot_p = tot.w;
    if (slot < s.B) {
      seg_off[slot] = seg;
      int base = seg;
      for (int w = 0; w < NW; ++w) {
        const int t = lds_tbl[w * s.B + slot];
        lds_tbl[w * s.B + slot] = base;
        base += t;
      }
      if (is_small) tasks[sb] = make_int4(slot, seg, n, -1);
      else
        for (int j = 0; j < nt; ++j)
          tasks[task_room - 1 - (tb + j)] = make_int4(slot, seg + j * kTaskChunk, min(kTaskChunk, n - j * kTaskChunk) | (is_multi ? mb << kTaskCountBits : 0),
                                                      is_multi ? part_base + pb + j : -1);
      if (is_multi) multi[mb] = make_int4(n, part_base + pb, nt, 0);
    }
    seg_carry += tot_n;
    small_carry += tot_s;
    task_carry += tot_t;
    multi_carry += tot_m;
    part_carry += tot_p;
  }
  if (threadIdx.x == 0) {
    seg_off[s.B] = seg_carry | (multi_carry > 0 ? kSomeSlotIsSplit : 0);
    c.n_tasks[(unit * sh.batch + b) * 2] = small_carry;
    c.n_tasks[(unit * sh.batch + b) * 2 + 1] = task_carry;
  }
  __syncthreads();

  // pass 2: write the members, ascending inside every slot
  int *members_dst = lds_members ? lds_members : members;
  if (wave < NW) {
    for (int i0 = r0; i0 < r1; i0 += 64 * kCsrAhead) {
      int slotv[kCsrAhead], keptv[kCsrAhead];
#pragma unroll
      for (int u = 0; u < kCsrAhead; ++u) {
        const int i = i0 + 64 * u + lane;
        slotv[u] = i < r1 ? assign[i] : -1;
      }
#pragma unroll
      for (int u = 0; u < kCsrAhead; ++u) keptv[u] = slotv[u] >= 0 ? kept[slotv[u]] : -1;
#pragma unroll
      for (int u = 0; u < kCsrAhead; ++u) {
        if (i0 + 64 * u >= r1) break;
        const int i = i0 + 64 * u + lane, slot = slotv[u];
        const bool member = slot >= 0 && keptv[u] != i;
        int below, total;
        same_slot_rank(member, slot, nbits, below, total);
        if (member) {
          const int cur = lds_tbl[wave * s.B + slot];
          members_dst[cur + below] = i;
          if (below == 0) lds_tbl[wave * s.B + slot] = cur + total;
        }
      }
    }
  }
  if (lds_members) {
    __syncthreads();
    for (int i = threadIdx.x; i < seg_carry; i += kCsrThreads) members[i] = members_dst[i];
  }
}

}  // namespace flowmm
