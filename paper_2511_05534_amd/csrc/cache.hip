// Decode-time maintenance of the compacted cache: the cache-append equation of the paper's
// Preliminary section, K_t = [K_{t-1}, k_t], V_t = [V_{t-1}, v_t], on a cache that keeps head room
// for decoded tokens behind every sequence's merged prompt rows, and the copy that puts the rows of
// a re-merge back at the head of the sequence's range.  Pure data movement in 16-byte chunks.
#include "device_common.h"
#include "kernels.h"
#include "profile.h"

namespace flowmm {

namespace {

// grid (sequences of this launch, kv heads, layers); one thread per 16-byte chunk of the K row and of the V row
template <int N, int NCH>
__global__ __launch_bounds__(64) void cache_append_kernel(AppendArgs<N> a) {
  const int b = blockIdx.x, g = blockIdx.y, l = blockIdx.z;
  const int t = threadIdx.x;
  if (t >= 2 * NCH) return;
  const int tensor = t / NCH, ch = t % NCH;
  const long long dst_row = (long long)l * a.ks_layer + (long long)g * a.ks_head + (long long)a.row[b] * a.ks_tok;
  const long long src_row = (((long long)l * gridDim.y + g) * a.batch + b) * NCH;
  const uint4 *src = reinterpret_cast<const uint4 *>(tensor ? a.v_new : a.k_new);
  uint4 *dst = reinterpret_cast<uint4 *>(tensor ? a.V_c : a.K_c);
  dst[dst_row + ch] = src[src_row + ch];
}

// Merge of one sequence's rows in place: row s of the range becomes the mean of its pivot's row kept[s] and its
// members' rows.  One workgroup per (part of the channels, tensor, kv head, layer): NCH 16-byte
// chunks of every row; the parts know nothing of each other.  The pivots ascend, so kept[s] >= s and a pivot's
// row lies behind every row written before it has been read; the members' rows, which may lie anywhere, wait
// in LDS.  The slots are taken kSlots at a time: all pivot rows of a round have arrived (barrier) before its first
// row is written, and the next round's rows (all behind this round's) are on their way meanwhile.
// Bound by HBM: rows and members read once, merged rows written once, where merging beside the cache and copying
// back moves every merged row three times (256 units x 1023 rows back to 819: 109 -> 50 us).
constexpr int kInPlaceThreads = 512;
constexpr int kInPlaceRows = 4;  // rows in flight per lane group
// A slot of more than kTaskChunk members is added up kRunOfSlot members at a time by as many lane groups as it has of these, before the slots are taken in turn:
// one lane group alone takes 80 ns a member (a re-merge of 8 units x 2400 rows, 2000 of them into one slot, 243 -> 85 us; beside the cache 93).  The sums
// of the runs, and then the slot's, take the place of its first members.  (And no longer chain of fp32 roundings than a task beside the cache has: a single one over the 2300
// members that fit LDS in shares of 64 bytes could be off by 2^-13.)
constexpr int kRunOfSlot = 32;

template <bool BF16, int NCH>
__global__ __launch_bounds__(kInPlaceThreads, 4) void merge_in_place_kernel(InPlaceArgs a) {
  constexpr int EPC = BF16 ? 8 : 4, U = kInPlaceRows;
  constexpr int kGroups = kInPlaceThreads / NCH, kSlots = kGroups * U;
  typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) u32x4_t lds_rows[];  // [members][NCH], then kept [B], member offsets [B + 1], runs of long slots (number, then
  // the first member of each, a slot's first run with the slot's members above 16 bits)
  const int tensor = blockIdx.x & 1, gkv = blockIdx.y, l = blockIdx.z;
  const long long unit = (long long)l * gridDim.y + gkv;
  const int rg = threadIdx.x / NCH, ch = threadIdx.x % NCH;
  int *lds_kept = reinterpret_cast<int *>(lds_rows + a.max_members * NCH), *lds_seg = lds_kept + a.B, *lds_runs = lds_seg + a.B + 1;
  u32x4_t *rows = reinterpret_cast<u32x4_t *>(tensor ? a.V_c : a.K_c) + (long long)l * a.ks_layer + (long long)gkv * a.ks_head + (blockIdx.x >> 1) * NCH + ch;
  const int *kept = a.kept_idx + unit * a.B, *seg = a.seg_off + unit * (a.B + 1), *members = a.members + unit * a.T;
  const int n_members = seg[a.B] & ~kSomeSlotIsSplit;
  const bool long_slots = (seg[a.B] & kSomeSlotIsSplit) != 0;
  for (int i = threadIdx.x; i < a.B; i += kInPlaceThreads) {
    lds_kept[i] = kept[i];
    lds_seg[i] = seg[i];
  }
  if (threadIdx.x == 0) lds_seg[a.B] = n_members;
  for (int i0 = rg; i0 < n_members; i0 += kSlots) {
    u32x4_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = rows[(long long)members[min(i0 + u * kGroups, n_members - 1)] * a.ks_tok];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * kGroups < n_members) lds_rows[(i0 + u * kGroups) * NCH + ch] = v[u];
  }
  __syncthreads();
  auto add_member = [&](int m, float (&acc)[EPC]) {
    float f[EPC];
    uint4 w;
    const u32x4_t r = lds_rows[m * NCH + ch];
    __builtin_memcpy(&w, &r, 16);
    chunk_to_floats<BF16>(w, f);
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] += f[e];
  };
  auto add_parked = [&](int m, float (&acc)[EPC]) {
    float sum[EPC];
    __builtin_memcpy(sum, lds_rows + m * NCH + ch, 16);
    if constexpr (BF16) __builtin_memcpy(sum + 4, lds_rows + (m + 1) * NCH + ch, 16);
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] += sum[e];
  };
  if (__builtin_expect(long_slots, 0)) {
    if (threadIdx.x == 0) lds_runs[0] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < a.B; i += kInPlaceThreads) {
      const int m0 = lds_seg[i], m1 = lds_seg[i + 1];
      if (m1 - m0 <= kTaskChunk) continue;
      int at = 1 + atomicAdd(lds_runs, (m1 - m0) / kRunOfSlot);
      lds_runs[at] = m0 | (m1 - m0) << 16;
      for (int m = m0 + kRunOfSlot; m + kRunOfSlot <= m1; m += kRunOfSlot) lds_runs[++at] = m;
    }
    __syncthreads();
    const int n_runs = lds_runs[0];
    auto park = [&](int m, const float (&acc)[EPC]) {
      __builtin_memcpy(lds_rows + m * NCH + ch, acc, 16);
      if constexpr (BF16) __builtin_memcpy(lds_rows + (m + 1) * NCH + ch, acc + 4, 16);
    };
    for (int i = rg; i < n_runs; i += kGroups) {
      const int m = lds_runs[1 + i] & 0xffff;
      float acc[EPC] = {};
#pragma unroll 4
      for (int j = 0; j < kRunOfSlot; ++j) add_member(m + j, acc);
      park(m, acc);
    }
    __syncthreads();
    for (int i = rg; i < n_runs; i += kGroups) {
      const int n = lds_runs[1 + i] >> 16, m0 = lds_runs[1 + i] & 0xffff;
      if (n == 0) continue;
      float acc[EPC] = {};
      int m = m0;
      for (; m + kRunOfSlot <= m0 + n; m += kRunOfSlot) add_parked(m, acc);
      for (; m < m0 + n; ++m) add_member(m, acc);
      park(m0, acc);
    }
    __syncthreads();
  }
  auto request = [&](int s0, u32x4_t (&v)[U]) {  // the pivot rows of the round at slot s0 (the last one's again past the end)
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = rows[(long long)lds_kept[min(s0 + u * kGroups + rg, a.B - 1)] * a.ks_tok];
  };
  u32x4_t cur[U], next[U];
  request(0, cur);
  for (int s0 = 0; s0 < a.B; s0 += kSlots) {
    // this round's rows are there; the U stores of the round before may still be on their way
    if (s0 == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(U) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");  // the builtin alone does not keep the compiler from moving stores above it
    if (s0 + kSlots < a.B) request(s0 + kSlots, next);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int slot = s0 + u * kGroups + rg;
      if (slot < a.B) {
        const int m0 = lds_seg[slot], m1 = lds_seg[slot + 1];
        u32x4_t out = cur[u];
        if (m1 > m0) {
          float acc[EPC];
          uint4 w;
          __builtin_memcpy(&w, &out, 16);
          chunk_to_floats<BF16>(w, acc);
          if (__builtin_expect(long_slots && m1 - m0 > kTaskChunk, 0)) add_parked(m0, acc);
          else
            for (int m = m0; m < m1; ++m) add_member(m, acc);
          const float den = (float)(1 + m1 - m0);
#pragma unroll
          for (int e = 0; e < EPC; ++e) acc[e] = acc[e] / den;
          w = floats_to_chunk<BF16>(acc);
          __builtin_memcpy(&out, &w, 16);
        }
        rows[(long long)slot * a.ks_tok] = out;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = next[u];
  }
}

// grid (row groups, kv heads, layers): rows [0, B) of the dense [Lyr][Hkv][B][d] source go to rows
// [row0, row0 + B) of the strided cache
__global__ __launch_bounds__(256) void cache_store_rows_kernel(StoreRowsArgs a) {
  const int g = blockIdx.y, l = blockIdx.z;
  const long long chunks = (long long)a.B * a.nch;
  const uint4 *srcK = reinterpret_cast<const uint4 *>(a.K_src) + ((long long)l * gridDim.y + g) * chunks;
  const uint4 *srcV = reinterpret_cast<const uint4 *>(a.V_src) + ((long long)l * gridDim.y + g) * chunks;
  uint4 *dstK = reinterpret_cast<uint4 *>(a.K_c) + (long long)l * a.ks_layer + (long long)g * a.ks_head + (long long)a.row0 * a.ks_tok;
  uint4 *dstV = reinterpret_cast<uint4 *>(a.V_c) + (long long)l * a.ks_layer + (long long)g * a.ks_head + (long long)a.row0 * a.ks_tok;
  for (long long q = (long long)blockIdx.x * 256 + threadIdx.x; q < chunks; q += (long long)gridDim.x * 256) {
    const long long s = q / a.nch;
    const int ch = (int)(q - s * a.nch);
    dstK[s * a.ks_tok + ch] = srcK[q];
    dstV[s * a.ks_tok + ch] = srcV[q];
  }
}

template <int N>
hipError_t launch_append_n(const AppendCall &c, const int *cu_capacity, const int *lengths, int b0, int n, int Hkv, int n_layers, hipStream_t stream) {
  AppendArgs<N> a;
  const long long first = (long long)b0 * c.nch * 16;
  a.K_c = c.K_c; a.V_c = c.V_c;
  a.k_new = reinterpret_cast<const char *>(c.k_new) + first; a.v_new = reinterpret_cast<const char *>(c.v_new) + first;
  a.ks_layer = c.ks_layer; a.ks_head = c.ks_head; a.ks_tok = c.ks_tok; a.batch = c.batch;
  for (int i = 0; i < N; ++i) a.row[i] = i < n ? cu_capacity[b0 + i] + lengths[b0 + i] : 0;
  const dim3 grid(n, Hkv, n_layers);
  ProfScope ps(stream, KID_CACHE_APPEND);
  switch (c.nch) {
    case 8: cache_append_kernel<N, 8><<<grid, 64, 0, stream>>>(a); break;
    case 16: cache_append_kernel<N, 16><<<grid, 64, 0, stream>>>(a); break;
    default: cache_append_kernel<N, 32><<<grid, 64, 0, stream>>>(a); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_cache_append(const AppendCall &c, const int *cu_capacity, const int *lengths, int Hkv, int n_layers, hipStream_t stream) {
  for (int b0 = 0; b0 < c.batch; b0 += kAppendSeqs) {
    const int n = c.batch - b0 < kAppendSeqs ? c.batch - b0 : kAppendSeqs;
    const hipError_t e = n <= kAppendSeqsSmall ? launch_append_n<kAppendSeqsSmall>(c, cu_capacity, lengths, b0, n, Hkv, n_layers, stream)
                                               : launch_append_n<kAppendSeqs>(c, cu_capacity, lengths, b0, n, Hkv, n_layers, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

namespace {

template <bool BF16, int NCH>
hipError_t launch_in_place_t(const InPlaceArgs &a, int parts, int Hkv, int n_layers, size_t lds, hipStream_t stream) {
  const hipError_t e = allow_full_lds<merge_in_place_kernel<BF16, NCH>>();
  if (e != hipSuccess) return e;
  ProfScope ps(stream, KID_MERGE_IN_PLACE);
  merge_in_place_kernel<BF16, NCH><<<dim3(2 * parts, Hkv, n_layers), kInPlaceThreads, lds, stream>>>(a);
  return hipGetLastError();
}

template <bool BF16>
hipError_t launch_in_place_by_width(const InPlaceArgs &a, int nch, int parts, int Hkv, int n_layers, size_t lds, hipStream_t stream) {
  switch (nch / parts) {
    case 4: return launch_in_place_t<BF16, 4>(a, parts, Hkv, n_layers, lds, stream);
    case 8: return launch_in_place_t<BF16, 8>(a, parts, Hkv, n_layers, lds, stream);
    case 16: return launch_in_place_t<BF16, 16>(a, parts, Hkv, n_layers, lds, stream);
    default: return launch_in_place_t<BF16, 32>(a, parts, Hkv, n_layers, lds, stream);
  }
}

size_t in_place_lds(const Shape &sh, int parts) {
  return (size_t)sh.maxE * sh.d * (sh.bf16 ? 2 : 4) / parts + (2 * (size_t)sh.maxB + 1) * sizeof(int);
}

// Into how many parts of their channels a unit's rows are cut for the merge in place; 0: merged beside the cache and copied back, as is what does not
// fit LDS (member rows: about 1200 shares of 128 bytes) and the weighted merge, whose V rows need the K rows.
// A workgroup keeps as much in flight whatever its share of a row: two parts where that doubles the workgroups that the chip holds at once and one
// part leaves it fewer than one and a half a compute unit (224 units x 1503 of 1716 rows, 448 workgroups or 896: 207, 206).  A re-merge, beside ->
// one part, two, us: 256 units x 819 of 1023 rows of 256 bytes 185 -> 142, 144; x 2600 of 3500 741 -> -, 691; 1024 x 1200 of 1600 930 -> 816, 739;
// 640 x 700 of 1050 413 -> 363, 309; 112 x 900 of 1100 120 -> 106, 99; 112 x 3200 of 3700 (two parts: 448 workgroups, one to a compute unit) 446 -> 396, 415; 64 x 2000 of 2300 206 -> 207, 187.
// Shares of less than a line of 128 bytes only where the chip has a compute unit for each; two parts -> four: 256 x 819 144 -> 166, 48 x 1500 142 -> 145, 32 x 1800 of
// 2100 155 -> 150, 4 x 400 of 500 49.1 -> 46.9.  With fewer units the kernels that spread a unit over workgroups win for long ones; beside -> here: 48
// units x 3000 301 -> 293; 32 x 1800 153 -> 150, x 2600 209 -> 209; 16 x 600 57.0 -> 55.8, x 1500 124.5 -> 127.7; 4 x 400 48.5 -> 46.9, x 1000 63.9 -> 67.0.
int in_place_parts(const Shape &sh) {
  if (sh.batch != 1 || sh.unit_path || sh.weighted_merge) return 0;
  constexpr int kUnitsOfChip = 256;  // compute units
  const long long units = (long long)sh.n_layers * sh.Hkv, row = (long long)sh.d * (sh.bf16 ? 2 : 4);
  int parts = 0;
  long long at_once = 0;
  for (int p = 1; row / p >= 64; p *= 2) {
    const size_t lds = in_place_lds(sh, p);
    if (lds > kLdsBytes - 1024) continue;
    const long long wgs = 2 * units * p;
    if (row / p < 128 && wgs > kUnitsOfChip) break;
    const long long per_cu = kLdsBytes / (long long)lds < 4 ? kLdsBytes / (long long)lds : 4;
    const long long now = wgs < kUnitsOfChip * per_cu ? wgs : kUnitsOfChip * per_cu;
    if (parts && (2 * at_once >= 3 * kUnitsOfChip || now < 2 * at_once)) break;
    parts = p;
    at_once = now;
  }
  if (!parts) return 0;
  return units >= 48 || sh.maxB * row / parts <= (units >= 32 ? 128 : 40) * 1024 ? parts : 0;
}

}  // namespace

bool merge_in_place_fits(const Shape &sh) { return in_place_parts(sh) > 0; }

hipError_t launch_merge_in_place(const Ctx &c, void *K_c, void *V_c) {
  const Shape &sh = c.sh;
  InPlaceArgs a;
  a.K_c = K_c; a.V_c = V_c;
  a.ks_layer = sh.ks_layer; a.ks_head = sh.ks_head; a.ks_tok = sh.ks_tok;
  a.kept_idx = c.kept_idx; a.seg_off = c.seg_off; a.members = c.members;
  a.T = sh.T; a.B = sh.SB; a.max_members = sh.maxE;
  const int parts = in_place_parts(sh), nch = sh.d * (sh.bf16 ? 2 : 4) / 16;
  const size_t lds = in_place_lds(sh, parts) + (1 + (size_t)sh.maxE / kRunOfSlot) * sizeof(int);  // (within the 1024 bytes that in_place_parts leaves)
  return sh.bf16 ? launch_in_place_by_width<true>(a, nch, parts, sh.Hkv, sh.n_layers, lds, c.stream)
                 : launch_in_place_by_width<false>(a, nch, parts, sh.Hkv, sh.n_layers, lds, c.stream);
}

hipError_t launch_cache_store_rows(const StoreRowsArgs &a, int Hkv, int n_layers, hipStream_t stream) {
  const long long chunks = (long long)a.B * a.nch;
  const int gx = (int)((chunks + 255) / 256 < 64 ? (chunks + 255) / 256 : 64);
  ProfScope ps(stream, KID_CACHE_STORE_ROWS);
  cache_store_rows_kernel<<<dim3(gx > 0 ? gx : 1, Hkv, n_layers), 256, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace flowmm
