// Device code shared by the bf16 attention kernels (flash.hip, flash64.hip): tiles of 64 rows of a head in LDS, filled by loads straight
// from global memory, the two kinds of fragment reads, conversions.
#pragma once
#include "nn.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;

// 2^x as the bare hardware instruction: results below the smallest normal number flush to zero, which is what a
// probability that small is worth; the library routine's extra range handling costs five more instructions per value
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// two floats to a packed pair of bf16, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ bf16x8 pack8(const f32x16 &v, int r0) {
  u32x4 u = {pack2(v[r0], v[r0 + 1]), pack2(v[r0 + 2], v[r0 + 3]), pack2(v[r0 + 4], v[r0 + 5]), pack2(v[r0 + 6], v[r0 + 7])};
  return __builtin_bit_cast(bf16x8, u);
}

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

// Causal work per query (or key) block grows linearly with its index, and all workgroups of a launch are
// usually resident at once, two per CU (workgroup b and b + half land on the same CU).  Blocks are therefore
// handed out in "snake" order: the first half of the grid takes the items from the most expensive down, the
// second half from the cheapest up, so that the two workgroups sharing a CU add up to the same work.
// Returns the rank of this workgroup's item in the list sorted by decreasing work.
__device__ __forceinline__ int snake_rank(int b, int nwg) {
  const int half = nwg >> 1;
  return b < half ? b : nwg - 1 - (b - half);
}

template <int DH>
struct Geo {
  static constexpr int KS = DH / 16, MT = DH / 32, RB = DH * 2;  // k-steps and 32-column blocks of a head, bytes of a row
  static constexpr int TILE_B = 64 * RB;                         // one staged tile
  static constexpr int STAGE_B = 2 * TILE_B;                     // K and V (or Q and dO)
  static constexpr int CPR = DH / 8, RPP = 64 / CPR;             // 16-byte chunks of a row, rows in a one-KB piece
  static __device__ __forceinline__ int swz(int r) {
    return DH == 128 ? 4 * (r & 3) + ((r >> 2) & 3) : DH == 64 ? 4 * ((r >> 1) & 1) + ((r >> 2) & 3) : (r >> 2) & 3;
  }
};
typedef __attribute__((address_space(3))) void *lds_void;

// Per-lane byte offsets (within a tile) of the two kinds of fragment reads.
template <int DH>
struct ReadOffsets {
  using G = Geo<DH>;
  uint32_t fo[G::KS];             // plain fragment of k-step ks for tile row (lane & 31); add 32 RB per 32 rows
  uint32_t ta[G::MT], tb[G::MT];  // transposing reads of head-dim block i: contraction rows +0..3 and +8..11; add 16 RB per 16 rows
  __device__ __forceinline__ void init(int lane) {
    const int c = lane & 31, g = lane >> 5, s16 = lane & 15, rho = (s16 >> 2) & 3, dlt = (s16 & 3) >> 1, hi = (lane >> 4) & 1;
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) fo[ks] = (uint32_t)(c * G::RB + (((2 * ks + g) ^ G::swz(c)) << 4));
    const int within = (s16 & 1) * 8, ra = 4 * g + rho, rb = ra + 8;
#pragma unroll
    for (int i = 0; i < G::MT; ++i) {
      ta[i] = (uint32_t)(ra * G::RB + within + (((4 * i + 2 * hi + dlt) ^ G::swz(ra)) << 4));
      tb[i] = (uint32_t)(rb * G::RB + within + (((4 * i + 2 * hi + dlt) ^ G::swz(rb)) << 4));
    }
  }
};

__device__ __forceinline__ bf16x8 frag(const char *tile, uint32_t off) { return *reinterpret_cast<const bf16x8 *>(tile + off); }
__device__ __forceinline__ bf16x8 frag_tr(const char *rows, uint32_t a, uint32_t b) {
  typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
  s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(rows + a));
  s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(rows + b));
  s16x8 v = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// Loads from global memory straight into LDS (lane l writes its 16 or 4 bytes at lds + bytes * l; lanes whose offset
// is outside the descriptor's range write zeros).  Written as assembly on purpose: for the builtin form the compiler
// cannot tell which LDS bytes a load fills and makes every later transposing LDS read wait for ALL such loads in
// flight, which turns the prefetch of the next tile into a stall.  Completion is awaited explicitly (DL_WAIT_VM0
// followed by a barrier) before any wave reads the bytes.  M0 (the LDS base of the instruction) is saved and restored.
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
template <int BYTES>
__device__ __forceinline__ void dma(desc_t desc, const char *lds, uint32_t voff) {
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void)(lds));
  uint32_t keep;
  if (BYTES == 16)
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "s"(l), "v"(voff), "s"(desc) : "memory");
  else
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dword %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "s"(l), "v"(voff), "s"(desc) : "memory");
}

// Each of 4 waves brings in a quarter of a tile's one-KB pieces.
template <int DH>
struct TileLoader {
  using G = Geo<DH>;
  static constexpr int NP = G::TILE_B / 4096;
  uint32_t off[NP];  // byte offset of this lane's chunk within tile 0, from the buffer base
  __device__ __forceinline__ void init(int64_t ld_elems, uint32_t col_byte0, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int row = G::RPP * (wave + 4 * i) + lane / G::CPR, chunk = (lane % G::CPR) ^ G::swz(row);
      off[i] = (uint32_t)(row * ld_elems * 2) + col_byte0 + chunk * 16;
    }
  }
  __device__ __forceinline__ void issue(desc_t rsrc, char *dst, uint32_t tile_byte0, int wave) const {
#pragma unroll
    for (int i = 0; i < NP; ++i) dma<16>(rsrc, dst + (wave + 4 * i) * 1024, off[i] + tile_byte0);
  }
};

#define DL_WAIT_VM0 __builtin_amdgcn_s_waitcnt(0x0f70)
#define DL_WAIT_LGKM0 __builtin_amdgcn_s_waitcnt(0xc07f)

// Backward of the rotary embedding on a lane's gradient values of one row (acc[i][4 j + e] is head-dim column
// 32 i + 8 j + 4 g + e): columns f and f + DH/2 form a pair rotated by the angle of (position, f); the backward pass turns
// the gradient by the opposite angle.  tab holds (cos, sin) for f = 0 .. DH/2 - 1 of every position, DH floats per position.
template <int DH>
__device__ __forceinline__ void rope_grad(f32x16 (&acc)[Geo<DH>::MT], const float *tab, int pos, int g) {
  const f32x4 *row = reinterpret_cast<const f32x4 *>(tab + (int64_t)pos * DH);
#pragma unroll
  for (int v = 0; v < DH / 16; ++v) {  // the lane's groups of four consecutive pair indices
    const int f = 8 * v + 4 * g, v2 = v + DH / 16;  // group v of columns is registers 4 (v % 4) .. + 3 of block v / 4
    const f32x4 w0 = row[f / 2], w1 = row[f / 2 + 1];
    const float cs[4] = {w0[0], w0[2], w1[0], w1[2]}, sn[4] = {w0[1], w0[3], w1[1], w1[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = acc[v / 4][4 * (v % 4) + e], b = acc[v2 / 4][4 * (v2 % 4) + e];
      acc[v / 4][4 * (v % 4) + e] = a * cs[e] + b * sn[e];
      acc[v2 / 4][4 * (v2 % 4) + e] = b * cs[e] - a * sn[e];
    }
  }
}

}  // namespace
