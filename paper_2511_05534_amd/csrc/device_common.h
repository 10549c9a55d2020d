// Device-side helpers shared by the gfx950 kernels: MFMA fragments read straight from global
// memory or LDS in 16-byte chunks, wave64 reductions, and metadata look-ups.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <stddef.h>

#include "kernels.h"
#include "layout.h"

namespace flowmm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

// A row of head_dim elements is NCH 16-byte chunks.  In every contraction lane (n, half) of a
// wave (n = lane & 31, half = lane >> 5) owns the chunks 2t+half, t = 0..NF-1, of row n of
// its operand tile, so both operands of an MFMA see the same channel in the same k slot.
template <bool BF16, int D>
struct Cfg {
  static constexpr int kElemBytes = BF16 ? 2 : 4;
  static constexpr int NCH = D * kElemBytes / 16;  // chunks per row
  static constexpr int NF = NCH / 2;               // fragments per lane per row
  static constexpr int kElemsPerChunk = 16 / kElemBytes;
};

// acc[m][n] += sum over the chunk's channels of a(row m) * b(row n); 32x32 tile, lane holds
// column n = lane & 31 and rows m = 8*(i/4) + 4*(lane>>5) + (i%4), i = 0..15.
template <bool BF16>
__device__ __forceinline__ void mma_chunk(f32x16_t &acc, const uint4 &a, const uint4 &b) {
  if constexpr (BF16) {
    bf16x8_t av, bv;
    __builtin_memcpy(&av, &a, 16);
    __builtin_memcpy(&bv, &b, 16);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
  } else {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  }
}

// ---- fp32 contractions on the bf16 matrix cores ------------------------------------------------------------
// An fp32 number is the sum of three bf16 terms, each the rounding of what the terms before it leave.  Of the nine products of two numbers' terms the six
// largest are taken; the others are below 2^-26 of the product.  16 channels of a 32x32 tile are 192 cycles of matrix core instead of 512 (the fp32
// instructions run at a sixteenth of the rate), and 32x32x16 adds fewer partial sums: against 64 bits the products are closer than
// the fp32 instructions' (2-norm of the error over that of the products, 64 and 128 channels, fp32 instructions -> this: N(0,1) rows 1.5e-7 -> 1.1e-7 and
// 2.0e-7 -> 1.6e-7; 0.5 + 0.8 N(0,1) 1.2e-7 -> 0.9e-7 and 1.7e-7 -> 1.4e-7; log-normal magnitudes over e^6 8.2e-8 -> 7.3e-8 and 8.8e-8 ->
// 4.5e-8; one channel that all rows share 1.7e-7 -> 1.3e-7 and 2.6e-7 -> 2.1e-7).
// Two things the terms cannot hold.  A number beyond the largest bf16 (infinities and NaN among them) and a product of terms that overflows, also where the
// product of the numbers does not (1.8411e19 squared: both lead with 2^64), leave an infinity or a NaN in the accumulator.  A number below 2^-110 has terms
// below the smallest subnormal bf16: each of its products is off by up to 2^-134 of the other factor.  A tile with an infinity or a NaN, or one of whose
// rows in registers consists of such small numbers (at 2^-120 its products would be off by 3e-5 of themselves), is contracted again by the fp32
// instructions, whose result it then is.  Single small numbers, and the rows that stream past, are not looked for: they show only against factors above 2^100.
struct Split8 { bf16x8_t t[3]; };  // eight channels (a lane's two consecutive chunks)

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  const bf16x2_t p = __builtin_convertvector(f32x2_t{a, b}, bf16x2_t);
  unsigned u;
  __builtin_memcpy(&u, &p, 4);
  return u;
}

__device__ __forceinline__ Split8 split8(const uint4 &c0, const uint4 &c1) {
  float x[8] = {__uint_as_float(c0.x), __uint_as_float(c0.y), __uint_as_float(c0.z), __uint_as_float(c0.w),
                __uint_as_float(c1.x), __uint_as_float(c1.y), __uint_as_float(c1.z), __uint_as_float(c1.w)};
  Split8 s;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    unsigned w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      w[j] = pack_bf16(x[2 * j], x[2 * j + 1]);
      x[2 * j] -= __uint_as_float(w[j] << 16);
      x[2 * j + 1] -= __uint_as_float(w[j] & 0xffff0000u);
    }
    __builtin_memcpy(&s.t[k], w, 16);
  }
  return s;
}

__device__ __forceinline__ void mma_split8(f32x16_t &acc, const Split8 &a, const Split8 &b) {  // the small terms first
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[2], b.t[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[0], b.t[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[1], b.t[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[1], b.t[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[0], b.t[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.t[0], b.t[0], acc, 0, 0, 0);
}

// A row of this lane's as a matrix operand in registers: its NF fragments as they are, or (fp32) split into terms, for every use again or once for all
enum Operand { kPlain, kSplitEachTime, kSplitOnce };

// infinity if a lane's part of its row is smaller than 2^-110 throughout (and not 0), else 0
template <int NF>
__device__ __forceinline__ float too_small_to_split(const uint4 (&raw)[NF]) {
  float most = 0.f;
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    most = __builtin_elementwise_maximum(most, __builtin_elementwise_maximum(fabsf(__uint_as_float(raw[i].x)), fabsf(__uint_as_float(raw[i].y))));
    most = __builtin_elementwise_maximum(most, __builtin_elementwise_maximum(fabsf(__uint_as_float(raw[i].z)), fabsf(__uint_as_float(raw[i].w))));
  }
  return __any(most > 0.f && most < 0x1p-110f) ? INFINITY : 0.f;
}

template <int NF, Operand HOW>
struct RowOperand {
  uint4 f[NF];
  float small = 0.f;
  __device__ __forceinline__ void set(const uint4 (&raw)[NF]) {
#pragma unroll
    for (int i = 0; i < NF; ++i) f[i] = raw[i];
    if constexpr (HOW != kPlain) small = too_small_to_split(raw);
  }
  __device__ __forceinline__ Split8 pair(int p) {
    // (opaque: terms kept from one use to the next would take the registers that this saves)
    asm volatile("" : "+v"(f[2 * p].x), "+v"(f[2 * p].y), "+v"(f[2 * p].z), "+v"(f[2 * p].w), "+v"(f[2 * p + 1].x), "+v"(f[2 * p + 1].y), "+v"(f[2 * p + 1].z), "+v"(f[2 * p + 1].w));
    return split8(f[2 * p], f[2 * p + 1]);
  }
};
template <int NF>
struct RowOperand<NF, kSplitOnce> {
  Split8 s[NF / 2];
  float small;
  __device__ __forceinline__ void set(const uint4 (&raw)[NF]) {
    small = too_small_to_split(raw);
#pragma unroll
    for (int p = 0; p < NF / 2; ++p) s[p] = split8(raw[2 * p], raw[2 * p + 1]);
  }
  __device__ __forceinline__ const Split8 &pair(int p) const { return s[p]; }
};

// acc[j] = products of the rows in regs[j], j = 0 .. NJ - 1, with the row whose fragment f is frag(f) (fp32); REGS_FIRST: the rows in registers are the tile's
// rows, else its columns.  raw(j, f): fragment f of the row in regs[j] as it is in memory.  kPlain: by the fp32 instructions.
template <bool REGS_FIRST, int NF, Operand HOW, int NJ, class Frag, class Raw>
__device__ __forceinline__ void f32_products(f32x16_t (&acc)[NJ], RowOperand<NF, HOW> *regs, Frag frag, Raw raw) {
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
  if constexpr (HOW == kPlain) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const uint4 o = frag(f);
#pragma unroll
      for (int j = 0; j < NJ; ++j) mma_chunk<false>(acc[j], REGS_FIRST ? regs[j].f[f] : o, REGS_FIRST ? o : regs[j].f[f]);
    }
    return;
  } else {
#pragma unroll
    for (int p = 0; p < NF / 2; ++p) {
      const Split8 o = split8(frag(2 * p), frag(2 * p + 1));
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if constexpr (REGS_FIRST) mma_split8(acc[j], regs[j].pair(p), o);
        else mma_split8(acc[j], o, regs[j].pair(p));
        if constexpr (HOW == kSplitEachTime) __builtin_amdgcn_sched_barrier(0);  // one pair's terms at a time
      }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      float most = regs[j].small;  // (NaN where one of them is)
#pragma unroll
      for (int i = 0; i < 16; i += 2) most = __builtin_elementwise_maximum(most, __builtin_elementwise_maximum(fabsf(acc[j][i]), fabsf(acc[j][i + 1])));
      if (__any(!(most < INFINITY))) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
#pragma unroll 1
        for (int f = 0; f < NF; ++f) {
          const uint4 a = raw(j, f), b = frag(f);
          mma_chunk<false>(acc[j], REGS_FIRST ? a : b, REGS_FIRST ? b : a);
        }
      }
    }
  }
}

__device__ __forceinline__ int acc_row(int i, int half) { return 8 * (i >> 2) + 4 * half + (i & 3); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// round-to-nearest-even float -> bf16 bits (finite inputs; NaN stays NaN)
__device__ __forceinline__ uint32_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

template <bool BF16>
__device__ __forceinline__ void chunk_to_floats(const uint4 &c, float *f) {
  if constexpr (BF16) {
    f[0] = bf16_bits_to_float(c.x & 0xffffu); f[1] = bf16_bits_to_float(c.x >> 16);
    f[2] = bf16_bits_to_float(c.y & 0xffffu); f[3] = bf16_bits_to_float(c.y >> 16);
    f[4] = bf16_bits_to_float(c.z & 0xffffu); f[5] = bf16_bits_to_float(c.z >> 16);
    f[6] = bf16_bits_to_float(c.w & 0xffffu); f[7] = bf16_bits_to_float(c.w >> 16);
  } else {
    f[0] = __uint_as_float(c.x); f[1] = __uint_as_float(c.y);
    f[2] = __uint_as_float(c.z); f[3] = __uint_as_float(c.w);
  }
}

template <bool BF16>
__device__ __forceinline__ uint4 floats_to_chunk(const float *f) {
  uint4 c;
  if constexpr (BF16) {
    c.x = float_to_bf16_bits(f[0]) | (float_to_bf16_bits(f[1]) << 16);
    c.y = float_to_bf16_bits(f[2]) | (float_to_bf16_bits(f[3]) << 16);
    c.z = float_to_bf16_bits(f[4]) | (float_to_bf16_bits(f[5]) << 16);
    c.w = float_to_bf16_bits(f[6]) | (float_to_bf16_bits(f[7]) << 16);
  } else {
    c.x = __float_as_uint(f[0]); c.y = __float_as_uint(f[1]);
    c.z = __float_as_uint(f[2]); c.w = __float_as_uint(f[3]);
  }
  return c;
}

template <bool BF16>
__device__ __forceinline__ float chunk_sumsq(const uint4 &c) {
  float f[8];
  chunk_to_floats<BF16>(c, f);
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < (BF16 ? 8 : 4); ++j) s = fmaf(f[j], f[j], s);
  return s;
}

// sum of squares of a chunk added to s; bf16 pairs go through the two-element dot product instruction
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
template <bool BF16>
__device__ __forceinline__ float chunk_sumsq_acc(const uint4 &c, float s) {
  if constexpr (BF16) {
    const unsigned w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bf16x2_t v;
      __builtin_memcpy(&v, &w[j], 4);
      s = __builtin_amdgcn_fdot2_f32_bf16(v, v, s, false);
    }
    return s;
  } else {
    return s + chunk_sumsq<false>(c);
  }
}

// 1 / sqrt(sum of squares), 0 for a zero row.  Candidates of the match compare at 2^-19 relative resolution, so a last bit here decides
// ties: every kernel that matches takes its norms from this function, over sums in the order of group_sum.
__device__ __forceinline__ float inverse_norm(float ss) { return ss > 0.f ? 1.0f / sqrtf(ss) : 0.f; }

// running (max, sum of exp2) pairs of a softmax row, in the log2 domain
__device__ __forceinline__ void stat_combine(float &m, float &z, float m2, float z2) {
  const float M = fmaxf(m, m2);
  if (M == -INFINITY) { m = M; z = 0.f; return; }
  z = z * fast_exp2(m - M) + z2 * fast_exp2(m2 - M);
  m = M;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sum over the LPR lanes that share a row, left in every one of them, in the order of a tree of exchanges between lanes LPR / 2, .., 2, 1
// apart (bit for bit: an addition's operands may change places), by DPP operands on the vector unit: the halves of 32 lanes swap, inside a row of 16
// lanes a rotation brings what the exchange would, and 8 lanes shift by four, up or down, then permute inside their quads.
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(LPR == 8 || LPR == 16 || LPR == 32, "rows of 8, 16 or 32 chunks");
  if constexpr (LPR == 32) {
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  if constexpr (LPR == 8) {
    int far = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x104, 0xf, 0x5, false);               // row_shl:4 into lanes 0..3 of the 8
    far = __builtin_amdgcn_update_dpp(far, __float_as_int(v), 0x114, 0xf, 0xa, false);                 // row_shr:4 into lanes 4..7
    v += __int_as_float(far);
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4e, 0xf, 0xf, false));   // quad_perm:[2,3,0,1]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, false));   // quad_perm:[1,0,3,2]
  } else {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));  // row_ror:8
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));  // row_ror:4
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));  // row_ror:2
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));  // row_ror:1
  }
  return v;
}

// Direct global -> LDS load: lane i of the wave fetches BYTES (4 or 16) bytes from base + byte_off
// (base wave-uniform, in scalar registers; the lane's part is a 32-bit offset, so no lane keeps a
// 64-bit address) and they land at lds_base + i * BYTES (lds_base wave-uniform).  Lanes that are
// switched off leave their bytes alone.  Issued as inline assembly so that the compiler does not
// wait for it before unrelated LDS reads (it cannot tell two LDS buffers apart); the statement
// sets M0 and says so in its clobber list (the compiler keeps M0 out of register allocation and
// warns about any such entry; the entry is still what orders its own M0 writes around this one).
// The caller waits with s_waitcnt vmcnt(0) and a barrier before reading the data.
typedef __attribute__((address_space(3))) void lds_void;
template <int BYTES>
__device__ __forceinline__ void load_to_lds(const void *base, unsigned byte_off, void *lds_base) {
  static_assert(BYTES == 4 || BYTES == 16, "one dword or four per lane");
  const unsigned lds_addr = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void *)lds_base);
  // the base goes through the first lane's copy of it: free when it already sits in scalar registers,
  // and it keeps the operand a scalar pair when the compiler has lost track of its uniformity
  const unsigned long long bits = (unsigned long long)(uintptr_t)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)bits), hi = __builtin_amdgcn_readfirstlane((unsigned)(bits >> 32));
  base = reinterpret_cast<const void *>((uintptr_t)(((unsigned long long)hi << 32) | lo));
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr) : "memory", "m0");
#pragma clang diagnostic pop
}

// Rows of one (sequence, kv head, layer) by token, as 16-byte chunks; a row that is not wanted comes as zeros and costs no traffic.
// NEAR: the rows lie within 4 GiB: buffer loads, whose lanes past the end of the range read zeros.  No load is under a branch then, so
// that all of a trip are on their way together (behind a branch the compiler has to wait for the loads before it as soon as it
// uses one of them: the rows of a trip of four came in two to three round trips).
template <bool NEAR>
struct RowSource;
template <>
struct RowSource<true> {
  __amdgpu_buffer_rsrc_t rsrc;
  unsigned stride, lane_off;  // bytes
  __device__ __forceinline__ RowSource(const void *base, long long ks_tok, int L, int nch, int ch) {
    // (uniform: the descriptor sits in scalar registers)
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)(unsigned)(((L - 1) * ks_tok + nch) * 16), 0x00020000);
    stride = (unsigned)ks_tok * 16u;
    lane_off = (unsigned)ch * 16u;
  }
  typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
  // where the lane's chunk of a row lies: the same in the K and the V rows, which share their strides
  __device__ __forceinline__ unsigned at(int tok, bool wanted) const {
    unsigned off = (unsigned)tok * stride + lane_off;
    asm volatile("" : "+v"(off));  // (keeps the choice below a select: as a branch it brings the waits back)
    return wanted ? off : 0xfffffff0u;  // (the range is a multiple of 16 below 2^32)
  }
  __device__ __forceinline__ u32x4_t raw_chunk(unsigned off) const { return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0); }
  __device__ __forceinline__ u32x4_t raw_row(int tok, bool wanted) const { return raw_chunk(at(tok, wanted)); }
  __device__ __forceinline__ uint4 chunk(unsigned off) const {
    const u32x4_t v = raw_chunk(off);
    return make_uint4(v[0], v[1], v[2], v[3]);
  }
  __device__ __forceinline__ uint4 row(int tok, bool wanted) const { return chunk(at(tok, wanted)); }
};
template <>
struct RowSource<false> {
  const uint4 *base;
  long long ks_tok;
  __device__ __forceinline__ RowSource(const void *b, long long ks, int, int, int ch) : base(reinterpret_cast<const uint4 *>(b) + ch), ks_tok(ks) {}
  __device__ __forceinline__ uint4 row(int tok, bool wanted) const { return wanted ? base[(long long)tok * ks_tok] : make_uint4(0, 0, 0, 0); }
};

// The rows of 32 tokens as MFMA operand fragments (this lane's chunks 2t+half of row n), fetched as
// whole rows.  Asked for straight from memory, those fragments make every load instruction touch 32
// cache lines for 32 bytes each, and a compute unit's L1 looks up one line per clock: 16 bytes per
// clock, and the waves wait at their load instructions meanwhile.  Here the wave fetches whole rows
// (64/NCH rows per instruction, every line touched once) into a staging area of its own in LDS with
// direct global->LDS loads; the chunk a lane asks for is chosen so that the chunks of row r land
// XOR-swizzled by r, and the fragments are then read from there without bank conflicts.
//   base  : wave-uniform; row t starts at base + t * row_stride chunks (32-bit byte offsets: the
//           caller has checked that the rows lie within 4 GiB of base)
//   tok   : the row this lane's fragments belong to (lanes n and n + 32 pass the same)
//   stage : 32 * NCH chunks of LDS that no other wave touches until the call has returned
template <bool BF16, int D>
__device__ __forceinline__ void request_rows_staged(const void *base, unsigned row_stride, int tok, uint4 *stage) {
  constexpr int NCH = Cfg<BF16, D>::NCH;
  static_assert(NCH <= 64 && (NCH & (NCH - 1)) == 0, "rows of a power-of-two number of chunks");
  constexpr int RPI = 64 / NCH;  // rows per load instruction
  const int lane = threadIdx.x & 63;
  const int rl = lane / NCH, slot = lane % NCH;
#pragma unroll
  for (int j = 0; j < 32 / RPI; ++j) {
    const int r = j * RPI + rl;
    const int t = __shfl(tok, r, 64);
    const int ch = slot ^ (r & (NCH - 1));
    load_to_lds<16>(base, ((unsigned)t * row_stride + (unsigned)ch) * 16u, stage + j * 64);
  }
}

// The fragments of the rows that request_rows_staged asked for (waits for this wave's outstanding loads
// first; only this wave reads the area, so no barrier), and a wait for the reads themselves: on return
// the area may be written again.
template <bool BF16, int D>
__device__ __forceinline__ void read_rows_staged(const uint4 *stage, uint4 (&frag)[Cfg<BF16, D>::NF]) {
  constexpr int NCH = Cfg<BF16, D>::NCH, NF = Cfg<BF16, D>::NF;
  const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
  __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
  for (int f = 0; f < NF; ++f) frag[f] = stage[n * NCH + ((2 * f + half) ^ (n & (NCH - 1)))];
  __builtin_amdgcn_s_waitcnt(0);
}

template <bool BF16, int D>
__device__ __forceinline__ void fetch_rows_staged(const void *base, unsigned row_stride, int tok, uint4 *stage,
                                                  uint4 (&frag)[Cfg<BF16, D>::NF]) {
  request_rows_staged<BF16, D>(base, row_stride, tok, stage);
  read_rows_staged<BF16, D>(stage, frag);
}

// lane number, computed where it stands: what follows from it is cheap and is not kept in registers
// across the loop around it
__device__ __forceinline__ int lane_id_here() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}

// A tile of key rows in LDS that direct global->LDS loads fill (whole rows, 1 KB = kGroup rows per load
// instruction) and that is read as MFMA fragments (lane n: a chunk of row n) without bank conflicts: the
// chunks of a row are XOR-permuted by its place in the group and every group is followed by a few chunks of
// padding, so that one chunk column of 16 consecutive rows falls on 16 different 16-byte columns of the banks.
// The permutation touches the two low bits of the chunk number only: a lane needs two base addresses, for
// even and odd fragments, and everything else is an immediate offset.
template <bool BF16, int D>
struct KeyTile {
  static constexpr int NCH = Cfg<BF16, D>::NCH;
  static_assert(NCH == 8 || NCH == 16 || NCH == 32, "rows of 128, 256 or 512 bytes");
  static constexpr int kGroup = 64 / NCH;
  static constexpr int kGroupChunks = 64 + (NCH == 32 ? 2 : 4);
  static constexpr int kRows = NCH == 32 ? 64 : 128;
  static constexpr int kChunks = kRows / kGroup * kGroupChunks;
  __device__ static __forceinline__ int permute(int row_in_group) { return NCH == 8 ? row_in_group >> 1 : row_in_group; }
  // bytes from a tile's start to chunk 2 * odd + half of row n (n < 32); fragment f of block kb of 32 rows lies
  // block_bytes(kb) + 64 * (f >> 1) behind frag_offset(n, half, f & 1)
  __device__ static __forceinline__ int frag_offset(int n, int half, int odd) {
    return ((n / kGroup) * kGroupChunks + (n % kGroup) * NCH + ((2 * odd + half) ^ permute(n % kGroup))) * 16;
  }
  static constexpr int block_bytes(int kb) { return kb * (32 / kGroup) * kGroupChunks * 16; }
  // this wave's share (one of WAVES) of the rows r0 .. r0 + kRows - 1 of src (row 0 at src, row stride in chunks),
  // clamped to row `last`
  template <int WAVES>
  __device__ static __forceinline__ void request(const uint4 *src, long long row_stride, int r0, int last, uint4 *tile, int wave) {
    const int lane = lane_id_here(), j = lane / NCH;
    const int ch = (lane % NCH) ^ permute(j);
    constexpr int kLoads = kRows / kGroup;
    static_assert(kLoads % WAVES == 0, "every wave asks for as many groups");
    const uint4 *base = src + r0 * row_stride;
    if (row_stride < (1ll << 32) / (16 * kRows)) {
#pragma unroll
      for (int i = 0; i < kLoads / WAVES; ++i) {
        const int g = i * WAVES + wave;
        const int r = min(g * kGroup + j, last - r0);
        load_to_lds<16>(base, ((unsigned)r * (unsigned)row_stride + (unsigned)ch) * 16u, tile + g * kGroupChunks);
      }
    } else {  // rows too far apart for 32-bit byte offsets
      for (int i = 0; i < kLoads / WAVES; ++i) {
        const int g = i * WAVES + wave;
        const int r = min(g * kGroup + j, last - r0);
        tile[g * kGroupChunks + lane] = base[r * row_stride + ch];
      }
    }
  }
};

// For grids whose x extent counts sequences (or a fixed number of workgroups per sequence) and whose
// y, z are kv head and layer: workgroups go to the eight XCDs in turn by their linear index, so a
// batch of eight would pin each sequence, long ones included, to one XCD.  Rotating x by the other
// two coordinates spreads every sequence over all XCDs; for fixed (y, z) it is still a bijection.
__device__ __forceinline__ int rotated_block_x() { return (blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x; }

// Workgroups are handed to the eight XCDs in turn.  Of `total` pieces of work (a (layer, kv head) unit's `per_unit` pieces one after the other) every
// XCD gets an eighth in a row: nearly all of a unit's pieces share an L2, and all XCDs have as much to do whatever the number of units (with a unit
// to an XCD 20 units left four of the eight with three units each, the others with two: calls of 20 x 12000 tokens 218 -> 181 us, of 36 x 4000 121 -> 107).  False for the workgroups that round the grid up.
__device__ __forceinline__ bool xcd_share(int total, int per_unit, int &unit, int &piece) {
  const int share = (total + 7) >> 3, k = blockIdx.x >> 3, i = (int)(blockIdx.x & 7) * share + k;
  if (k >= share || i >= total) return false;
  unit = i / per_unit;
  piece = i - unit * per_unit;
  return true;
}

// words that no kernel of the launch writes, read by scalar loads at wave-uniform indexes
typedef const __attribute__((address_space(4))) int *ScalarInts;
__device__ __forceinline__ ScalarInts scalar_ints(const int *p) { return (ScalarInts)(uintptr_t)p; }

// The metadata words for the first kernel of a call: in its own arguments (KernelArgs<A>, the kernel's only parameter) where they fit, else the
// workspace's, put there by a launch of their own.  Everything here is read by scalar loads.
template <class A>
__device__ __forceinline__ ScalarInts first_meta(const KernelArgs<A> &k, const int *in_workspace) {
  const ScalarInts args = (ScalarInts)__builtin_amdgcn_kernarg_segment_ptr();
  return k.meta.n > 0 ? args + offsetof(KernelArgs<A>, meta.w) / 4 : scalar_ints(in_workspace);
}

// sequence that owns flat index x given an increasing cumulative table cu[0..batch]
template <class Ints>
__device__ __forceinline__ int find_seq(Ints cu, int batch, int x) {
  int lo = 0, hi = batch;  // invariant: cu[lo] <= x < cu[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

struct SeqInfo {
  int tok_off, L, B, kept_off, win_has_img, n_text;
  float tau;
};

template <class Ints>
__device__ __forceinline__ SeqInfo load_seq(Ints meta, int b) {
  const Ints r = meta + meta[MW_OFF_SEQ] + b * SW_WORDS;
  SeqInfo s;
  s.tok_off = r[SW_TOK_OFF];
  s.L = r[SW_L];
  s.B = r[SW_B];
  s.kept_off = r[SW_KEPT_OFF];
  s.tau = __int_as_float(r[SW_TAU]);
  s.win_has_img = r[SW_WIN_HAS_IMG];
  s.n_text = r[SW_N_TEXT];
  return s;
}

// v / d and the remainder; inv = (2^32 - 1) / d makes the product's upper half the quotient or one less (scalar multiplications; a
// division by an unknown number costs a workgroup 0.2 us)
__device__ __forceinline__ unsigned quotient(unsigned v, unsigned d, unsigned inv, unsigned &rem) {
  unsigned q = (unsigned)(((unsigned long long)v * inv) >> 32);
  rem = v - q * d;
  if (rem >= d) { ++q; rem -= d; }
  return q;
}

// position inside the window of query row `row` of a kv head: the heads' windows of W rows lie next to each other
__device__ __forceinline__ int window_row(const Shape &sh, int row) {
  unsigned r;
  quotient((unsigned)row, (unsigned)sh.W, sh.inv_window, r);
  return (int)r;
}

// (sequence, kv head, layer) of a workgroup where the grid has one for each of them: (sequences, kv heads, layers).  Unequal sequences: the longest
// first, as a grid that ends with them waits for them (whole calls, the
// sequences of a head in turn -> this, us: 112 units x 8 of 2048 to 8192 tokens 1612 -> 1595, x 3 of up to 16384 859 -> 848, x 8 of up to 400
// 173 -> 170, 256 x 4 of up to 1000 332 -> 322; not in the unit path, whose merge has long streams cover the starts of short ones: 1024 x 4 of up
// to 600 332 and 340).
struct UnitBlock { int b, gkv, l; };
template <class Ints>
__device__ __forceinline__ UnitBlock unit_block(const Shape &sh, Ints meta) {
  UnitBlock u;
  if (sh.by_length) {
    const unsigned lin = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    unsigned unit, gkv;
    const int x = (int)quotient(lin, (unsigned)(sh.Hkv * sh.n_layers), sh.inv_units, unit);
    u.l = (int)quotient(unit, gridDim.y, sh.inv_heads, gkv);
    u.gkv = (int)gkv;
    u.b = meta[meta[MW_OFF_SEQ] + x * SW_WORDS + SW_BY_LENGTH];
  } else {
    u.b = rotated_block_x();
    u.gkv = blockIdx.y;
    u.l = blockIdx.z;
  }
  return u;
}

__device__ __forceinline__ SeqInfo inline_seq(const InlineMeta &m, int b) {
  SeqInfo s;
  s.tok_off = m.tok_off[b];
  s.L = m.L[b];
  s.B = m.B[b];
  s.kept_off = m.kept_off[b];
  s.tau = m.tau[b];
  s.win_has_img = (m.win_has_img >> b) & 1u;
  s.n_text = 0;
  return s;
}

// modality (0 text, 1 image) of position i of sequence b: the first span that ends after i.
// The loop runs over the spans of the sequence with wave-uniform bounds, so the span table is read
// with scalar loads (a per-lane walk would turn it into vector loads from the argument block, which
// then queue behind every outstanding key load).
__device__ __forceinline__ int inline_mod(const InlineMeta &m, int b, int i) {
  const int first = m.span_off[b], last = m.span_off[b + 1] - 1;
  int mod = (m.span_is_image >> last) & 1u;
  for (int j = last - 1; j >= first; --j)
    if (i < m.span_end[j]) mod = (m.span_is_image >> j) & 1u;
  return mod;
}

// modality of a position in [from, L) of sequence b, where few spans lie (from: wave-uniform)
__device__ __forceinline__ int late_modality(ScalarInts meta, int b, int from, int pos) {
  const ScalarInts rec = meta + meta[MW_OFF_SEQ] + b * SW_WORDS, spans = meta + meta[MW_OFF_SPANS];
  int j = rec[SW_SPAN_OFF] + rec[SW_N_SPANS] - 1, mod = spans[3 * j + 2];
  while (spans[3 * j] > from) {  // (the first span starts at 0)
    --j;
    mod = pos < spans[3 * j + 1] ? spans[3 * j + 2] : mod;
  }
  return mod;
}

// The modality span that an ascending stream of keys is in, walked with scalar loads (wave-uniform arguments).
struct SpanCursor {
  ScalarInts spans;
  int at, end;
  unsigned img;
  __device__ __forceinline__ SpanCursor(ScalarInts meta, int b) {
    spans = meta + meta[MW_OFF_SPANS];
    at = (meta + meta[MW_OFF_SEQ] + b * SW_WORDS)[SW_SPAN_OFF] - 1;
    end = 0;
    img = 0u;
  }
  // bit j: key key0 + j of the sequence is an image token (key0 < L, not below the last call's)
  __device__ __forceinline__ unsigned mask(int key0, int L) {
    while (end <= key0) {
      ++at;
      end = spans[3 * at + 1];
      img = spans[3 * at + 2] ? 0xffffffffu : 0u;
    }
    unsigned bits = img;
    if (end < key0 + 32) {
      bits &= (1u << (end - key0)) - 1u;
      for (int q = at + 1, e = end; e < min(key0 + 32, L); ++q) {
        if (spans[3 * q + 2]) bits |= 0xffffffffu << (e - key0);
        e = spans[3 * q + 1];
        if (e < key0 + 32) bits &= (1u << (e - key0)) - 1u;
      }
    }
    return bits;
  }
};

// What the kernels behind a call's first one read of the batch: the metadata words in the workspace, a modality byte per token and the tokens'
// places in their sequence's class order (all text positions ascending, then all image positions ascending).

// the tokens of span `at`, by a workgroup of THREADS
template <int THREADS, class Ints>
__device__ __forceinline__ void expand_span(Ints meta, int at, uint8_t *mod, int *cls_order) {
  const int batch = meta[MW_BATCH];
  const Ints spans = meta + meta[MW_OFF_SPANS] + 3 * at;
  // owner sequence: the one whose span range contains this span
  int b = 0;
  for (int i = 0; i < batch; ++i) {
    const Ints r = meta + meta[MW_OFF_SEQ] + i * SW_WORDS;
    if (at >= r[SW_SPAN_OFF] && at < r[SW_SPAN_OFF] + r[SW_N_SPANS]) b = i;
  }
  const Ints rec = meta + meta[MW_OFF_SEQ] + b * SW_WORDS;
  const int tok_off = rec[SW_TOK_OFF];
  const uint8_t m = (uint8_t)spans[2];
  int before = m ? rec[SW_N_TEXT] : 0;  // tokens of this class in earlier spans of the sequence
  for (int j = rec[SW_SPAN_OFF]; j < at; ++j) {
    const Ints sp = meta + meta[MW_OFF_SPANS] + 3 * j;
    if (sp[2] == m) before += sp[1] - sp[0];
  }
  for (int i = spans[0] + threadIdx.x; i < spans[1]; i += THREADS) {
    mod[tok_off + i] = m;
    cls_order[tok_off + before + i - spans[0]] = i;
  }
}

// Workgroup `at` behind the ones that do the first kernel's own work (there is one for every span where its arguments hold the words): a launch
// for this alone was 5 us of every call.
template <int THREADS>
__device__ __forceinline__ void place_meta(const Ctx &c, ScalarInts meta, int n_words, int at) {
  if (at == 0)
    for (int i = threadIdx.x; i < n_words; i += THREADS) c.meta[i] = meta[i];
  if (at < meta[MW_N_SPANS]) expand_span<THREADS>(meta, at, c.mod, c.cls_order);
}

}  // namespace flowmm
