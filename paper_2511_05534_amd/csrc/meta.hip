// Places the host-packed metadata words at the head of the workspace (they travel as kernel
// arguments, so no host memory has to outlive the call and nothing synchronises) and expands
// the modality spans into one byte per packed token: for calls whose words do not fit the arguments of their first
// kernel, which does both otherwise (place_meta).
#include "device_common.h"
#include "kernels.h"
#include "profile.h"

namespace flowmm {

namespace {

__global__ __launch_bounds__(256) void meta_upload_kernel(MetaChunk chunk, int *dst, int n) {
  for (int i = threadIdx.x; i < n; i += 256) dst[i] = chunk.w[i];
}

// one workgroup per span
__global__ __launch_bounds__(256) void expand_modality_kernel(const int *meta, uint8_t *mod, int *cls_order) {
  expand_span<256>(meta, blockIdx.x, mod, cls_order);
}

}  // namespace

hipError_t launch_meta_upload(const Ctx &c, const int *words, int n_words, bool expand_modality) {
  for (int off = 0; off < n_words; off += kMetaChunkWords) {
    MetaChunk chunk;
    const int n = n_words - off < kMetaChunkWords ? n_words - off : kMetaChunkWords;
    for (int i = 0; i < n; ++i) chunk.w[i] = words[off + i];
    ProfScope ps(c.stream, KID_META_UPLOAD);
    meta_upload_kernel<<<1, 256, 0, c.stream>>>(chunk, c.meta + off, n);
  }
  if (expand_modality) {
    ProfScope ps(c.stream, KID_EXPAND_MODALITY);
    expand_modality_kernel<<<words[MW_N_SPANS], 256, 0, c.stream>>>(c.meta, c.mod, c.cls_order);
  }
  return hipGetLastError();
}

}  // namespace flowmm
