// Device code shared by the bf16 projection kernels (gemm.hip, gemm_dl.hip): operand types, the epilogue's arguments, conversions.
#pragma once
#include "act.h"
#include "nn.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// two floats to a packed pair of bf16, round to nearest even, in one instruction (v_cvt_pk_bf16_f32): the same bits as f2bf for
// every finite value and infinity (the software form costs about eight instructions and a branch per value, which showed in
// the epilogue: 40.6 -> 39.9 ms per forward+backward pass)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

struct Ep {
  float alpha;
  const void *bias;
  const float *residual;
  void *out;
  int out_f32;
  int64_t ldc;
  void *act_out;  // f(out as stored) of an ungated activation, laid out like out, bf16 (or null); out may then be null
  int act;
  int vec_ok;  // out (and residual, act_out) rows allow 4-element vector accesses: ldc % 4 == 0, 16-byte aligned bases
};

// Weight gradients (TN products over the same contraction) that share a launch; tiles are numbered through all of them.
struct TnProduct {
  const uint16_t *a, *b;
  float *out;      // with a cut contraction: the product's part 0 in the scratch
  int64_t lda, ldb;
  int M, N, first, tiles_m, tiles_n;  // first: number of its first tile
  float alpha;
  int vec_ok;
};
struct TnGroup {
  int n;
  TnProduct p[kGroupProducts];
};
struct NoGroup {};
// the product that tile `bid` belongs to; bid becomes the tile's number within it
__device__ __forceinline__ int product_of(const TnGroup &g, int &bid) {
  int q = 0;
#pragma unroll
  for (int i = 1; i < kGroupProducts; ++i)
    if (i < g.n && bid >= g.p[i].first) q = i;
  bid -= g.p[q].first;
  return q;
}

constexpr uint32_t kOob = 0x80000000u;  // byte offset beyond every buffer: loads return 0, stores are dropped

// Elements from a panel's base to the end of its last 16-byte chunk.  A load that reaches beyond the buffer's range returns nothing at
// all, so the range has to include the whole of a last row's partly used chunk (the chunk is aligned and holds at least one
// element of the operand, so reading it is safe; what it holds beyond the operand meets zeros or is not stored).
__device__ __forceinline__ int64_t panel_span(int km, int64_t ld, int rows, int rows_left, int K) {
  const int64_t len = km ? K : rows_left, up = (len + 7) / 8 * 8;
  return (km ? (int64_t)(rows - 1) : (int64_t)(K - 1)) * ld + (up < ld ? up : ld);
}

typedef __attribute__((address_space(3))) void *lds_void;
typedef uint32_t desc_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ desc_t make_desc(const void *p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  desc_t d;
  d.x = __builtin_amdgcn_readfirstlane((uint32_t)a);
  d.y = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
  d.z = __builtin_amdgcn_readfirstlane(bytes);
  d.w = 0x00020000u;
  return d;
}
// 16 bytes per lane from global memory straight into LDS at lds + 16 lane (zeros where voff is outside the descriptor's range).  As
// assembly because for the builtin form the compiler makes every later transposing LDS read wait for all such loads in flight.
__device__ __forceinline__ void dma16(desc_t desc, const char *lds, uint32_t voff) {
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void)(lds));
  uint32_t keep;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
               : "=&s"(keep) : "s"(l), "v"(voff), "s"(desc) : "memory");
}

// Stores four consecutive columns ncol .. ncol + 3 of row m: out = (v4 + bias) alpha + residual (STREAM: past the caches), and (ACT) its activation
template <bool STREAM, bool ACT>
__device__ __forceinline__ void store_quad(const Ep &ep, void *outp, int m, int ncol, int N, const f32x4 &v4, const float (&bias)[4], bool vec) {
  const int64_t o = (int64_t)m * ep.ldc + ncol;
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (v4[e] + bias[e]) * ep.alpha;
  if (vec) {
    if (ep.residual) {
      const f32x4 rr = *reinterpret_cast<const f32x4 *>(ep.residual + o);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += rr[e];
    }
    if (ep.out_f32) {
      const f32x4 w = {v[0], v[1], v[2], v[3]};
      f32x4 *p = reinterpret_cast<f32x4 *>(static_cast<float *>(outp) + o);
      if (STREAM) __builtin_nontemporal_store(w, p);
      else *p = w;
    } else {
      const u32x2 w = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
      u32x2 *p = reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(outp) + o);
      if (ACT && !outp) {
      } else if (STREAM) {
        __builtin_nontemporal_store(w, p);
      } else {
        *p = w;
      }
      if (ACT && ep.act_out) {
        const float f[4] = {act_value<false>(ep.act, bf2f((uint16_t)w.x)), act_value<false>(ep.act, bf2f((uint16_t)(w.x >> 16))),
                            act_value<false>(ep.act, bf2f((uint16_t)w.y)), act_value<false>(ep.act, bf2f((uint16_t)(w.y >> 16)))};
        const u32x2 a = {pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3])};
        u32x2 *q = reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(ep.act_out) + o);
        if (STREAM) __builtin_nontemporal_store(a, q);
        else *q = a;
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (ncol + e >= N) break;
      float x = v[e];
      if (ep.residual) x += ep.residual[o + e];
      if (ep.out_f32) {
        static_cast<float *>(outp)[o + e] = x;
      } else {
        const uint16_t w = f2bf(x);
        if (!ACT || outp) static_cast<uint16_t *>(outp)[o + e] = w;
        if (ACT && ep.act_out) static_cast<uint16_t *>(ep.act_out)[o + e] = f2bf(act_value<false>(ep.act, bf2f(w)));
      }
    }
  }
}

}  // namespace
