// Host-side launchers of the gfx950 kernels.  Every launcher enqueues on ctx.stream and
// returns the hipError_t of the launch; none of them synchronises or allocates.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <initializer_list>

#include "layout.h"

namespace flowmm {

// LDS of a compute unit, and the most one workgroup may ask for (static plus dynamic)
constexpr size_t kLdsBytes = 160 * 1024;

// A kernel that wants more than 64 KB of dynamic LDS needs its cap raised first.  The cap belongs
// to the function (per device), not to a launch, so it is raised once per kernel and device to all the
// LDS there is beside the kernel's static share: no later call changes it, whatever shapes other
// host threads launch at the same time.  Kernels that one launcher chooses from are raised together, for one look-up of the device.
template <auto... Kernels>
hipError_t allow_full_lds() {
  constexpr int kMaxDevices = 64;
  static std::atomic<bool> done[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < kMaxDevices && done[dev].load(std::memory_order_acquire)) return hipSuccess;
  for (const void *kernel : {reinterpret_cast<const void *>(Kernels)...}) {
    hipFuncAttributes at;
    if ((e = hipFuncGetAttributes(&at, kernel)) != hipSuccess) return e;
    const size_t room = kLdsBytes > at.sharedSizeBytes ? kLdsBytes - at.sharedSizeBytes : 0;
    if ((e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)room)) != hipSuccess) return e;
  }
  if (dev >= 0 && dev < kMaxDevices) done[dev].store(true, std::memory_order_release);
  return hipSuccess;
}

struct Ctx {
  Shape sh;
  InlineMeta inl;  // sequences: of up to kInlineSeqs; spans: when sh.unit_path
  hipStream_t stream;
  int layer0, layers;  // the unit-resident kernels work on layers [layer0, layer0 + layers) per launch
  // inputs
  const void *K, *V, *Q;
  // plan buffers
  float *importance, *rho;
  int *mode, *kept_idx, *assign, *n_dropped;
  // outputs
  void *K_out, *V_out;
  // workspace regions
  int *meta;
  uint8_t *mod;        // [T]                             modality of every packed token
  int *cls_order;      // [T]                             per sequence: text positions ascending, then image positions
  float4 *part_stats;  // [Lyr][Hkv][tiles_score][R_pad]  (max, sum exp2 over text, over image keys) of each row over a run, or
                       //                                 as float2 (max, sum exp2)
  float *cross_part;   // [Lyr][Hkv][tiles_score]         cross-modal mass of a kv head's query rows over a run
  int *ev_list;        // [Lyr][Hkv][T]                   the tokens to be matched, per sequence in class order (text, then image)
  int *ev_n;           // [Lyr][Hkv][batch][2]            how many of either class (all in the first one in a cross-modal layer)
  int *pl_slot;        // [Lyr][Hkv][2*SBP]               eligible pivots per (sequence, token class): their slots, ascending
  int *pl_tok;         // [Lyr][Hkv][2*SBP]               their positions
  float *pl_w;         // [Lyr][Hkv][2*SBP]               1/norm of those pivots (0 for a zero row)
  int *pl_n;           // [Lyr][Hkv][batch][2]            list lengths, padded to multiples of 32
  uint4 *pack;         // [Lyr][Hkv][2*SBP][row chunks+1] their K rows, one chunk of padding after each
  int *seg_off;        // [Lyr][Hkv][SB + batch]          CSR offsets of the members of each slot, their number (with kSomeSlotIsSplit)
  int *members;        // [Lyr][Hkv][T]                   evicted tokens grouped by slot, ascending
  int4 *tasks;         // [Lyr][Hkv][tasks_total]         (slot, first member, count and split slot, partial index or -1); per sequence the
                       //                                 small ones from the front of its range, the others from the back
  int *n_tasks;        // [Lyr][Hkv][batch][2]            how many of either kind
  int4 *multi;         // [Lyr][Hkv][multi_total]         slots cut into several tasks: (members, first partial, number of partials, partials that are there)
  float *partials;     // [Lyr][Hkv][part_total][2][d]    fp32 partial row sums of K and V
  float *partial_w;    // [Lyr][Hkv][part_total]          weight sums of those partials (weighted merge)
};

// The metadata words of a call in the arguments of its first kernel (n = 0: they did not fit, the workspace has them).  A kernel's arguments
// may take 4 KB.
constexpr int kMetaArgWords = 720;
struct MetaArg {
  int n;
  int w[kMetaArgWords];
};
template <class A>
struct KernelArgs {
  A a;
  MetaArg meta;
};
// n words, or (n = 0) none
template <class A>
inline void fill_kernel_args(KernelArgs<A> &k, const A &a, const int *words, int n) {
  static_assert(sizeof(KernelArgs<A>) <= 4096, "kernel arguments");
  k.a = a;
  k.meta.n = n;
  for (int i = 0; i < n; ++i) k.meta.w[i] = words[i];
}

// arguments of the exact (all-query) flow ratio that are not part of a plan
struct FlowExactArgs {
  const void *Q;                          // [Lyr][Hq][T][d] queries of every prompt token
  long long qs_layer, qs_head, qs_tok;    // strides in 16-byte chunks
  float *part;                            // [Lyr][Hq][qblocks_total] sum of the rows' cross-modal shares per query block
  int qblocks_total;
  int wgs_total;                          // workgroups per (kv head, layer)
  int group;                              // units that the grid takes in turn
  float *rho;                             // [Lyr][batch]
  int *mode;                              // [Lyr][batch]
};
hipError_t launch_flow_exact(const Ctx &c, const FlowExactArgs &a, const int *words, int n_words);

// arguments of the decode-step attention over the compacted cache; the description of the sequences rides in them
constexpr int kDecodeSeqs = 64;  // sequences per launch
struct DecodeArgs {
  const void *q;               // [Lyr][Hq][batch][d]
  const void *K_c, *V_c;       // [Lyr][Hkv][SB][d] merged rows
  void *out;                   // [Lyr][Hq][batch][d]
  float *part;                 // [Lyr][Hq][tasks][d + 2] partial (weighted V, max, sum) of the sequences of several tasks
  int Hq, Hkv, G, SB, batch;
  float scale_log2e;
  int chunk, waves;            // slots per task (workgroup); waves of a workgroup (bf16)
  int b0, n_seqs, tasks;       // sequences b0 .. b0 + n_seqs - 1 of the batch are in this launch, cut into tasks
  int full;                    // tasks of `chunk` slots: first in the order of the tasks, before the sequences' rests, the longest first
  int mixed;                   // (layer, kv head) units whose tasks the grid takes unit by unit; those of the others go task by task (-1: in any order)
  unsigned inv_tasks, inv_last, inv_heads;  // (2^32 - 1) / the tasks, the units past `mixed`, the kv heads
  int g0;                      // first query head (inside its kv group) of the current launch
  int rest[kDecodeSeqs / 4];     // sequences that have a rest, the longest first, a byte each
  // First slot and first task of each of them (task: bits 0..15; where the order counts, in bits 16.. the first full one among the full ones).
  // A workgroup starts with a look in here: every 64-byte line of the arguments that it touches is a round trip of 0.2 us, so what it reads
  // of a sequence shares a line, for a small batch that of the whole search (16 units x 7 sequences 6.8 -> 6.5 us).
  struct Seq { int slot, task; };
  alignas(64) Seq cu[kDecodeSeqs + 1];
};
static_assert(offsetof(DecodeArgs, cu) % 64 == 0 && 8 * sizeof(DecodeArgs::Seq) <= 64, "seven sequences and the end in one line");
hipError_t launch_decode_attention(const Shape &sh, const int *budgets, DecodeArgs a, hipStream_t stream);

// cache append (decode-time maintenance): one new K and V row per sequence, (layer, kv head) by (layer, kv head).
// The target rows of N sequences ride in the kernel arguments.  Launches whose arguments stay below about 100 bytes
// take 2.8 us of host time on this part, larger ones 3.7 (measured from 32 to 1608 bytes): small batches get N = 8.
constexpr int kAppendSeqsSmall = 8, kAppendSeqs = 64;
template <int N>
struct AppendArgs {
  void *K_c, *V_c;               // the cache, addressed through the strides below (16-byte chunks)
  const void *k_new, *v_new;     // [Lyr][Hkv][batch][d] contiguous, from the first sequence of this launch on
  long long ks_layer, ks_head, ks_tok;
  int batch;                     // of the call
  int row[N];                    // cache row (token index) that the i-th sequence of the launch appends to
};
struct AppendCall {
  void *K_c, *V_c;
  const void *k_new, *v_new;
  long long ks_layer, ks_head, ks_tok;
  int nch, batch;                // chunks per row
};
hipError_t launch_cache_append(const AppendCall &a, const int *cu_capacity, const int *lengths, int Hkv, int n_layers, hipStream_t stream);

// rows of a dense [Lyr][Hkv][B][d] pair of tensors stored to cache rows [row0, row0 + B)
struct StoreRowsArgs {
  void *K_c, *V_c;
  const void *K_src, *V_src;
  long long ks_layer, ks_head, ks_tok;
  int nch, B, row0;
};
hipError_t launch_cache_store_rows(const StoreRowsArgs &a, int Hkv, int n_layers, hipStream_t stream);

// the merge of a single sequence whose result replaces the head of its rows (cache re-merge)
struct InPlaceArgs {
  void *K_c, *V_c;
  long long ks_layer, ks_head, ks_tok;     // 16-byte chunks
  const int *kept_idx, *seg_off, *members; // [unit][B], [unit][B + 1], [unit][T]
  int T, B, max_members;
};
bool merge_in_place_fits(const Shape &sh);
hipError_t launch_merge_in_place(const Ctx &c, void *K_c, void *V_c);  // after launch_merge_csr

constexpr int kMetaChunkWords = 960;
struct MetaChunk { int w[kMetaChunkWords]; };

hipError_t launch_meta_upload(const Ctx &c, const int *words, int n_words, bool expand_modality);
// row statistics, column sums.  n_words > 0: the first kernel of the call, which places the metadata for the others too
hipError_t launch_score(const Ctx &c, const int *words, int n_words);
bool score_stream_fits(const Shape &sh);  // what Shape::score_stream is set to
int score_resident_waves(const Shape &sh);  // what Shape::score_resident is set to
hipError_t launch_select(const Ctx &c);   // flow + top-B split
hipError_t launch_match(const Ctx &c);
bool select_match_fits(const Shape &sh);  // what Shape::select_match is set to where the unit path does not fit
hipError_t launch_select_match(const Ctx &c, bool with_csr);  // in place of launch_select, launch_match and (with_csr) launch_merge_csr
hipError_t launch_merge_csr(const Ctx &c, const int *words, int n_words);  // (words as above, without modalities)
hipError_t launch_merge(const Ctx &c, bool with_csr, const int *words = nullptr, int n_words = 0);    // CSR build (unless it is there already), task sums, combine

// unit-resident path (short prompts): one workgroup per (sequence, kv head, layer)
bool unit_path_fits(const Shape &sh);
bool unit_merge_fits(const Shape &sh);  // what Shape::unit_merge is set to where the unit path does not fit
// score, select and the cross-modal match of every unit; with_flow adds the launch that settles the
// layer strategies and matches the units of intra-modal layers again (the plan is then complete)
hipError_t launch_unit_plan(const Ctx &c, bool with_flow = true);
hipError_t launch_unit_flow_match(const Ctx &c);
// merge; with_flow: the same workgroups first do what launch_unit_flow_match does for their unit
hipError_t launch_unit_merge(const Ctx &c, bool with_flow = false);

// static LDS needs, used by the host to reject shapes that cannot be staged
size_t score_lds_limit_bytes(const Shape &sh, long long rows);  // of kernels with that many query rows
size_t merge_csr_lds_bytes(int max_budget);

}  // namespace flowmm
