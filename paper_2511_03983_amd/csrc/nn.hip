// Memory-bound kernels of the subnet training path: embedding, norms (Appendix A.1), rotary positions,
// activations, losses, reductions for bias / gain gradients, and the local optimizer steps.
// Activations and weights are fp32 or bf16 (template flag BF); all arithmetic is fp32.
#include "act.h"
#include "nn.h"

namespace {

constexpr int kT = 256;
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));

template <int BF> struct El;
template <> struct El<0> {
  using T = float;
  static __device__ __forceinline__ float ld(const void *p, int64_t i) { return static_cast<const float *>(p)[i]; }
  static __device__ __forceinline__ void st(void *p, int64_t i, float v) { static_cast<float *>(p)[i] = v; }
};
template <> struct El<1> {
  using T = uint16_t;
  static __device__ __forceinline__ float ld(const void *p, int64_t i) {
    return __uint_as_float((uint32_t) static_cast<const uint16_t *>(p)[i] << 16);
  }
  static __device__ __forceinline__ void st(void *p, int64_t i, float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) u = (u >> 16) | 0x40u;
    else { u += 0x7fffu + ((u >> 16) & 1u); u >>= 16; }
    static_cast<uint16_t *>(p)[i] = (uint16_t)u;
  }
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// block-wide sum for kT threads; result valid in every thread
__device__ __forceinline__ float block_sum(float v, float *sh) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}
__device__ __forceinline__ float block_max(float v, float *sh) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// four consecutive values of an operand
template <int BF>
__device__ __forceinline__ f32x4v ld4(const void *p, int64_t vec) {
  if (BF) {
    const u32x2v u = static_cast<const u32x2v *>(p)[vec];
    return f32x4v{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
  }
  return static_cast<const f32x4v *>(p)[vec];
}

// ------------------------------------------------------------------------------------------- embedding
// A wave per row of D, 4 columns a lane where rows allow it (VEC): what bounded the forward kernel was a 64-bit
// division per element: 8192 x 768 in bf16 26 -> 11 us.  The backward one is bound by its atomics (26 us either way).
template <int BF, bool VEC>
__global__ __launch_bounds__(kT) void embed_fwd_kernel(const int32_t *tok, const void *E, const void *P, float *x, int N, int D, int64_t T) {
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= T) return;
  const int64_t e = (int64_t)tok[t] * D, p = t % N * D, o = t * D;
  if (VEC) {
#pragma unroll 4
    for (int c = 4 * lane; c < D; c += 256) {
      f32x4v v = ld4<BF>(E, (e + c) >> 2);
      if (P) v += ld4<BF>(P, (p + c) >> 2);
      *reinterpret_cast<f32x4v *>(x + o + c) = v;
    }
  } else {
    for (int c = lane; c < D; c += 64) {
      float v = El<BF>::ld(E, e + c);
      if (P) v += El<BF>::ld(P, p + c);
      x[o + c] = v;
    }
  }
}

__global__ __launch_bounds__(kT) void embed_bwd_tok_kernel(const int32_t *tok, const float *dx, float *dE, int D, int64_t T) {
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= T) return;
  const int64_t e = (int64_t)tok[t] * D, o = t * D;
  for (int c0 = lane; c0 < D; c0 += 256) {
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = c0 + 64 * k < D ? dx[o + c0 + 64 * k] : 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c0 + 64 * k < D) atomicAdd(&dE[e + c0 + 64 * k], v[k]);
  }
}

__global__ __launch_bounds__(kT) void embed_bwd_pos_kernel(const float *dx, float *dP, int B, int N, int D) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;  // over N*D
  if (i >= (int64_t)N * D) return;
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += dx[(int64_t)b * N * D + i];
  dP[i] = s;
}

template <int BF>
__global__ __launch_bounds__(kT) void cast_in_kernel(const void *src, float *dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) dst[i] = El<BF>::ld(src, i);
}

// ------------------------------------------------------------------------------------------- norms
// one wave per row
template <int BF, int RMS>
__global__ __launch_bounds__(kT) void norm_fwd_kernel(const float *x, const void *w, const void *b, void *y, float *stats, int T, int D, float eps) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= T) return;
  const float *xr = x + (int64_t)row * D;
  float mean = 0.f;
  if (!RMS) {
    float s = 0.f;
    for (int c = lane; c < D; c += 64) s += xr[c];
    mean = wave_sum(s) / D;
  }
  float s2 = 0.f;
  for (int c = lane; c < D; c += 64) { float d = xr[c] - mean; s2 += d * d; }
  const float rstd = 1.0f / sqrtf(wave_sum(s2) / D + eps);
  for (int c = lane; c < D; c += 64) {
    float v = (xr[c] - mean) * rstd * El<BF>::ld(w, c);
    if (b) v += El<BF>::ld(b, c);
    El<BF>::st(y, (int64_t)row * D + c, v);
  }
  if (lane == 0) { stats[2 * row] = mean; stats[2 * row + 1] = rstd; }
}

template <int BF, int RMS>
__global__ __launch_bounds__(kT) void norm_bwd_dx_kernel(const void *dy, const float *x, const void *w, const float *stats, float *dx, int accumulate,
                                                          void *dxb, int T, int D) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= T) return;
  const float mean = stats[2 * row], rstd = stats[2 * row + 1];
  const float *xr = x + (int64_t)row * D;
  float c1 = 0.f, c2 = 0.f;
  for (int c = lane; c < D; c += 64) {
    float dz = El<BF>::ld(dy, (int64_t)row * D + c) * El<BF>::ld(w, c);
    float z = (xr[c] - mean) * rstd;
    c1 += dz;
    c2 += dz * z;
  }
  c1 = RMS ? 0.f : wave_sum(c1) / D;
  c2 = wave_sum(c2) / D;
  for (int c = lane; c < D; c += 64) {
    float dz = El<BF>::ld(dy, (int64_t)row * D + c) * El<BF>::ld(w, c);
    float z = (xr[c] - mean) * rstd;
    float g = rstd * (dz - c1 - z * c2);
    const int64_t i = (int64_t)row * D + c;
    if (accumulate) g += dx[i];
    dx[i] = g;
    if (dxb) El<BF>::st(dxb, i, g);
  }
}

constexpr int kChunkRows = 16;

// partial[chunk][0][c] = sum over the chunk's rows of dy*z ; partial[chunk][1][c] = sum of dy
template <int BF>
__global__ __launch_bounds__(64) void norm_bwd_dw_kernel(const void *dy, const float *x, const float *stats, float *partial, int T, int D) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  const int chunk = blockIdx.y;
  if (c >= D) return;
  const int r0 = chunk * kChunkRows, r1 = min(r0 + kChunkRows, T);
  float sw = 0.f, sb = 0.f;
  for (int r = r0; r < r1; ++r) {
    float g = El<BF>::ld(dy, (int64_t)r * D + c);
    float z = (x[(int64_t)r * D + c] - stats[2 * r]) * stats[2 * r + 1];
    sw += g * z;
    sb += g;
  }
  partial[((int64_t)chunk * 2) * D + c] = sw;
  partial[((int64_t)chunk * 2 + 1) * D + c] = sb;
}

// four consecutive values to an operand (bf16: round to nearest even); returns what was stored
template <int BF>
__device__ __forceinline__ f32x4v st4(void *p, int64_t vec, const f32x4v &o) {
  if (BF) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 lo = {o[0], o[1]}, hi = {o[2], o[3]};
    const u32x2v pk = {__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2)), __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2))};
    static_cast<u32x2v *>(p)[vec] = pk;
    return f32x4v{__uint_as_float(pk.x << 16), __uint_as_float(pk.x & 0xffff0000u), __uint_as_float(pk.y << 16), __uint_as_float(pk.y & 0xffff0000u)};
  }
  static_cast<f32x4v *>(p)[vec] = o;
  return o;
}

// Fused norm backward for rows of D <= NV * 256 elements, D a multiple of 4: one pass over dy and x yields dx (+= when accumulating), its
// activation-type copy, and this chunk's partial sums for the gain / bias gradients.  A wave owns a row at a time and
// a lane the same 4 NV columns of every row (vector v = lane + 64 k holds columns 4v .. 4v+3; those beyond D are read from the last one and
// count as zero), so the parameter sums stay in registers across the chunk's rows; the W waves' sums are combined through LDS.
// CS: the copy's column sums are formed as well (csum[chunk][D]): the bias gradients of the projection that the copy goes back into,
// which otherwise cost a launch and another pass over it (8192 x 768 bf16: 7.8 us beside this kernel's 20).
// W = 8 instead of 4 where the chunks are fewer than the CUs, so that a wave has two rows after one another, not four.
// Bound by memory where the chunks fill the chip (8192 x 2048 bf16: 54 us, 5 TB/s).  Widths that are no multiple of 256 ran two kernels
// with 2- and 4-byte loads (forward and backward, us): 4000 x 1304 bf16 52 -> 28, 4096 x 520 38 -> 26; fp32 2000 x 3400 95 -> 38.
template <int BF, int RMS, int NV, bool CS, int W, bool FULL>
__global__ __launch_bounds__(64 * W) void norm_bwd_fused_kernel(const void *dy, const float *x, const void *w, const float *stats, float *dx, int accumulate,
                                                                void *dxb, float *partial, float *csum, int T, int Dn) {
  const int D = FULL ? NV * 256 : Dn;
  __shared__ float red[(RMS ? 1 : 2) * W * NV * 256];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, d4 = D >> 2;
  const int r0 = blockIdx.x * kChunkRows, r1 = min(r0 + kChunkRows, T);
  auto on = [&](int k) { return FULL || lane + 64 * k < d4; };
  auto at = [&](int k) { return FULL ? lane + 64 * k : min(lane + 64 * k, d4 - 1); };
  f32x4v wv[NV], aw[NV], ab[NV], ac[CS ? NV : 1];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    wv[k] = ld4<BF>(w, at(k));
    aw[k] = f32x4v{0.f, 0.f, 0.f, 0.f};
    ab[k] = f32x4v{0.f, 0.f, 0.f, 0.f};
    if (CS) ac[CS ? k : 0] = f32x4v{0.f, 0.f, 0.f, 0.f};
  }
  for (int r = r0 + wave; r < r1; r += W) {
    const float mean = stats[2 * r], rstd = stats[2 * r + 1];
    const int64_t rv = (int64_t)r * d4;
    f32x4v g[NV], z[NV];
    float c1 = 0.f, c2 = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int v = at(k);
      g[k] = ld4<BF>(dy, rv + v);
      z[k] = (reinterpret_cast<const f32x4v *>(x)[rv + v] - mean) * rstd;
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        g[k][e] = on(k) ? g[k][e] : 0.f;
        z[k][e] = on(k) ? z[k][e] : 0.f;
      }
      aw[k] += g[k] * z[k];
      if (!RMS) ab[k] += g[k];
      g[k] *= wv[k];  // dz
#pragma unroll
      for (int e = 0; e < 4; ++e) { c1 += g[k][e]; c2 += g[k][e] * z[k][e]; }
    }
    c1 = RMS ? 0.f : wave_sum(c1) / D;
    c2 = wave_sum(c2) / D;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      if (!on(k)) continue;
      f32x4v o = rstd * (g[k] - c1 - z[k] * c2);
      f32x4v *dp = reinterpret_cast<f32x4v *>(dx) + rv + lane + 64 * k;
      if (accumulate) o += *dp;
      *dp = o;
      if (dxb) {
        const f32x4v kept = st4<BF>(dxb, rv + lane + 64 * k, o);
        if (CS) ac[CS ? k : 0] += kept;
      }
    }
  }
  constexpr int LD = NV * 256;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    *reinterpret_cast<f32x4v *>(&red[wave * LD + 4 * (lane + 64 * k)]) = aw[k];
    if (!RMS) *reinterpret_cast<f32x4v *>(&red[(W + wave) * LD + 4 * (lane + 64 * k)]) = ab[k];
  }
  __syncthreads();
  auto sum = [&](int first, int c) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) t += red[(first + i) * LD + c];
    return t;
  };
  for (int c = threadIdx.x; c < D; c += 64 * W) {
    partial[((int64_t)blockIdx.x * 2) * D + c] = sum(0, c);
    if (!RMS) partial[((int64_t)blockIdx.x * 2 + 1) * D + c] = sum(W, c);
  }
  if (CS) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) *reinterpret_cast<f32x4v *>(&red[wave * LD + 4 * (lane + 64 * k)]) = ac[CS ? k : 0];
    __syncthreads();
    for (int c = threadIdx.x; c < D; c += 64 * W) csum[(int64_t)blockIdx.x * D + c] = sum(0, c);
  }
}

// The same for rows of up to NV * 1024 elements: four waves share a row and a thread holds vectors t + 256 k of it, so that the registers still allow
// three waves per SIMD (one wave a row: 256 registers, one wave; 8192 x 4096 bf16 210 us, 112); the next row's loads run under this row's
// sums, and the parameter sums are whole where they are formed.
template <int BF, int RMS, int NV, bool CS>
__global__ __launch_bounds__(kT) void norm_bwd_wide_kernel(const void *dy, const float *x, const void *w, const float *stats, float *dx, int accumulate,
                                                           void *dxb, float *partial, float *csum, int T, int D) {
  __shared__ float sh[2][2][4];
  const int wave = threadIdx.x >> 6, d4 = D >> 2;
  const int r0 = blockIdx.x * kChunkRows, r1 = min(r0 + kChunkRows, T);
  f32x4v wv[NV], aw[NV], ab[NV], ac[CS ? NV : 1];
  int at[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    at[k] = min((int)threadIdx.x + kT * k, d4 - 1);
    wv[k] = ld4<BF>(w, at[k]);
    aw[k] = f32x4v{0.f, 0.f, 0.f, 0.f};
    ab[k] = f32x4v{0.f, 0.f, 0.f, 0.f};
    if (CS) ac[CS ? k : 0] = f32x4v{0.f, 0.f, 0.f, 0.f};
  }
  struct Row { f32x4v g[NV], x[NV], d[NV]; float mean, rstd; };
  auto load = [&](Row &q, int r) {
    const int64_t rv = (int64_t)r * d4;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      q.g[k] = ld4<BF>(dy, rv + at[k]);
      q.x[k] = reinterpret_cast<const f32x4v *>(x)[rv + at[k]];
      q.d[k] = accumulate ? reinterpret_cast<const f32x4v *>(dx)[rv + at[k]] : f32x4v{0.f, 0.f, 0.f, 0.f};
    }
    q.mean = stats[2 * r];
    q.rstd = stats[2 * r + 1];
  };
  Row q;
  load(q, r0);
  for (int r = r0; r < r1; ++r) {
    Row next = q;
    if (r + 1 < r1) load(next, r + 1);
    float c1 = 0.f, c2 = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const bool on = (int)threadIdx.x + kT * k < d4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g = on ? q.g[k][e] : 0.f, z = on ? (q.x[k][e] - q.mean) * q.rstd : 0.f;
        aw[k][e] += g * z;
        if (!RMS) ab[k][e] += g;
        q.g[k][e] = g * wv[k][e];  // dz
        q.x[k][e] = z;
        c1 += q.g[k][e];
        c2 += q.g[k][e] * z;
      }
    }
    c1 = RMS ? 0.f : wave_sum(c1);
    c2 = wave_sum(c2);
    if ((threadIdx.x & 63) == 0) { sh[r & 1][0][wave] = c1; sh[r & 1][1][wave] = c2; }
    __syncthreads();  // (two sets: the next row's writes do not meet this row's reads)
    c1 = RMS ? 0.f : (sh[r & 1][0][0] + sh[r & 1][0][1] + sh[r & 1][0][2] + sh[r & 1][0][3]) / D;
    c2 = (sh[r & 1][1][0] + sh[r & 1][1][1] + sh[r & 1][1][2] + sh[r & 1][1][3]) / D;
    const int64_t rv = (int64_t)r * d4;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      if ((int)threadIdx.x + kT * k >= d4) continue;
      const f32x4v o = q.rstd * (q.g[k] - c1 - q.x[k] * c2) + q.d[k];
      reinterpret_cast<f32x4v *>(dx)[rv + at[k]] = o;
      if (dxb) {
        const f32x4v kept = st4<BF>(dxb, rv + at[k], o);
        if (CS) ac[CS ? k : 0] += kept;
      }
    }
    q = next;
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    if ((int)threadIdx.x + kT * k >= d4) continue;
    f32x4v *p = reinterpret_cast<f32x4v *>(partial + (int64_t)blockIdx.x * 2 * D);
    p[at[k]] = aw[k];
    if (!RMS) p[d4 + at[k]] = ab[k];
    if (CS) reinterpret_cast<f32x4v *>(csum + (int64_t)blockIdx.x * D)[at[k]] = ac[CS ? k : 0];
  }
}

// out[c] = alpha * sum_k partial[k*stride + c].  A workgroup owns 16 columns; its 256 threads are 16 chunk slices x
// 16 columns, each summing every sixteenth chunk in ascending order; the slices are then added in order.
__global__ __launch_bounds__(kT) void reduce_partial_kernel(const float *partial, int64_t stride, int n_chunks, float alpha, float *out, int n) {
  __shared__ float sh[16][16];
  const int col = threadIdx.x & 15, slice = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + col;
  float s = 0.f;
  if (c < n)
    for (int k = slice; k < n_chunks; k += 16) s += partial[(int64_t)k * stride + c];
  sh[slice][col] = s;
  __syncthreads();
  if (slice == 0 && c < n) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += sh[i][col];
    out[c] = alpha * t;
  }
}

// the same reduction for a batch of buffers in one launch: blockIdx.y = item
constexpr int kReduceBatch = 64;
struct ColReduceArgs {
  ColReduce item[kReduceBatch];
};
__global__ __launch_bounds__(kT) void reduce_partial_batch_kernel(const ColReduceArgs a, int n_chunks) {
  __shared__ float sh[16][16];
  const ColReduce it = a.item[blockIdx.y];
  const int col = threadIdx.x & 15, slice = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + col;
  if (blockIdx.x * 16 >= it.n) return;  // uniform over the workgroup
  float s = 0.f;
  if (c < it.n)
    for (int k = slice; k < n_chunks; k += 16) s += it.partial[(int64_t)k * it.stride + c];
  sh[slice][col] = s;
  __syncthreads();
  if (slice == 0 && c < it.n) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += sh[i][col];
    it.out[c] = it.alpha * t;
  }
}

// ... where n and the stride are multiples of 4 and the partial sums 16-byte aligned: 4 columns a thread, 64 a workgroup, the same order of
// additions and eight loads in flight.  What bounded it: half lines of 64 bytes, one load of a thread at a time; 64 sums
// of 768 columns over 512 chunks 38 -> 23 us.
__global__ __launch_bounds__(kT) void reduce_partial_batch_vec_kernel(const ColReduceArgs a, int n_chunks) {
  __shared__ f32x4v sh[16][16];
  const ColReduce it = a.item[blockIdx.y];
  const int lane = threadIdx.x & 15, slice = threadIdx.x >> 4, c = 64 * blockIdx.x + 4 * lane;
  if (64 * (int)blockIdx.x >= it.n) return;  // uniform over the workgroup
  f32x4v s = {0.f, 0.f, 0.f, 0.f};
  if (c < it.n) {
    const float *p = it.partial + c;
    int k = slice;
    for (; k + 7 * 16 < n_chunks; k += 8 * 16) {
      f32x4v v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const f32x4v *>(p + (int64_t)(k + 16 * j) * it.stride);
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; k < n_chunks; k += 16) s += *reinterpret_cast<const f32x4v *>(p + (int64_t)k * it.stride);
  }
  sh[slice][lane] = s;
  __syncthreads();
  if (slice == 0 && c < it.n) {
    f32x4v t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) t += sh[i][lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) it.out[c + e] = it.alpha * t[e];
  }
}

template <int BF>
__global__ __launch_bounds__(64) void colsum_kernel(const void *src, int64_t ld, float *partial, int T, int n) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  const int chunk = blockIdx.y;
  if (c >= n) return;
  const int r0 = chunk * kChunkRows, r1 = min(r0 + kChunkRows, T);
  float s = 0.f;
  for (int r = r0; r < r1; ++r) s += El<BF>::ld(src, (int64_t)r * ld + c);
  partial[(int64_t)chunk * n + c] = s;
}
// the same sums where rows can be read 16 bytes at a time: a thread owns 8 (bf16) or 4 columns of a chunk and has all its loads in
// flight; tpc = threads per chunk.  8192 x 768 bf16: 7.8 us with 2-byte loads, 5.3 here.
template <int BF>
__global__ __launch_bounds__(kT) void colsum_vec_kernel(const void *src, int64_t ld, float *partial, int T, int n, int tpc, int64_t total) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int chunk = (int)(i / tpc), v = (int)(i - (int64_t)chunk * tpc), r0 = chunk * kChunkRows, rows = min(kChunkRows, T - r0);
  constexpr int PER = BF ? 8 : 4;
  const u4 *p = static_cast<const u4 *>(src) + (int64_t)r0 * (ld / PER) + v;
  u4 x[kChunkRows];
#pragma unroll
  for (int r = 0; r < kChunkRows; ++r) x[r] = r < rows ? p[r * (ld / PER)] : u4{0u, 0u, 0u, 0u};
  f4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
  for (int r = 0; r < kChunkRows; ++r) {
    if (BF) {
      lo += f4{__uint_as_float(x[r].x << 16), __uint_as_float(x[r].x & 0xffff0000u), __uint_as_float(x[r].y << 16), __uint_as_float(x[r].y & 0xffff0000u)};
      hi += f4{__uint_as_float(x[r].z << 16), __uint_as_float(x[r].z & 0xffff0000u), __uint_as_float(x[r].w << 16), __uint_as_float(x[r].w & 0xffff0000u)};
    } else {
      lo += __builtin_bit_cast(f4, x[r]);
    }
  }
  f4 *o = reinterpret_cast<f4 *>(partial + (int64_t)chunk * n) + v * (PER / 4);
  o[0] = lo;
  if (BF) o[1] = hi;
}

// ------------------------------------------------------------------------------------------- rotary
__global__ __launch_bounds__(kT) void rope_table_kernel(float *tab, int N, int half, int dh, float theta) {
  int i = blockIdx.x * kT + threadIdx.x;
  if (i >= N * half) return;
  int pos = i / half, f = i - pos * half;
  double ang = (double)pos * pow((double)theta, -2.0 * (double)f / (double)dh);
  tab[2 * i] = (float)cos(ang);
  tab[2 * i + 1] = (float)sin(ang);
}

// q and k heads of a fused [T, 3*Hs*dh] buffer, in place; pair (i, i + dh/2)
template <int BF>
__global__ __launch_bounds__(kT) void rope_kernel(void *qkv, const float *tab, int N, int Hs, int dh, float sign, int64_t total) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;  // over T * 2Hs * half
  if (i >= total) return;
  const int half = dh / 2;
  int f = (int)(i % half);
  int64_t r = i / half;
  int head = (int)(r % (2 * Hs));
  int64_t t = r / (2 * Hs);
  int pos = (int)(t % N);
  const float c = tab[2 * (pos * half + f)], s = sign * tab[2 * (pos * half + f) + 1];
  const int64_t base = t * (3 * (int64_t)Hs * dh) + (int64_t)head * dh + f;
  float a = El<BF>::ld(qkv, base), b = El<BF>::ld(qkv, base + half);
  El<BF>::st(qkv, base, a * c - b * s);
  El<BF>::st(qkv, base + half, b * c + a * s);
}

// ------------------------------------------------------------------------------------------- activations
__device__ __forceinline__ float sigmoidf(float x) { return 1.f / (1.f + __expf(-x)); }

// `keep` (may be null): the Masked-TwIST neuron mask of Section 4.1, y = M * f(x).  keep[b] < 0 marks FFN block b (of
// `unit` neurons) as masked: its activations, and in the backward kernels its pre-activation gradients, are zero.
template <int BF>
__global__ __launch_bounds__(kT) void act_fwd_kernel(int act, const void *gu, void *a, int F, int64_t total, const int32_t *keep, int unit) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int64_t t = i / F;
  const int c = (int)(i - t * F);
  float o;
  if (act == TWIST_ACT_SWIGLU) {
    float g = El<BF>::ld(gu, t * 2 * F + c), u = El<BF>::ld(gu, t * 2 * F + F + c);
    o = g * sigmoidf(g) * u;
  } else {
    o = act_value<BF == 0>(act, El<BF>::ld(gu, i));
  }
  if (keep && keep[c / unit] < 0) o = 0.f;
  El<BF>::st(a, i, o);
}

template <int BF>
__global__ __launch_bounds__(kT) void act_bwd_kernel(int act, const void *gu, const void *da, void *dgu, int F, int64_t total, const int32_t *keep, int unit) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int64_t t = i / F;
  const int c = (int)(i - t * F);
  const float d = (keep && keep[c / unit] < 0) ? 0.f : El<BF>::ld(da, i);
  if (act == TWIST_ACT_SWIGLU) {
    float g = El<BF>::ld(gu, t * 2 * F + c), u = El<BF>::ld(gu, t * 2 * F + F + c);
    float sg = sigmoidf(g);
    El<BF>::st(dgu, t * 2 * F + F + c, d * g * sg);
    El<BF>::st(dgu, t * 2 * F + c, d * u * (sg + g * sg * (1.f - sg)));
  } else {
    float u = El<BF>::ld(gu, i);
    El<BF>::st(dgu, i, d * (act == TWIST_ACT_RELU ? (u > 0.f ? 1.f : 0.f) : gelu_tanh_grad<BF == 0>(u)));
  }
}

// ------------------------------------------------------------------------------------------- losses
// one workgroup per row: logsumexp, row loss, then dlogits in place
template <int BF, bool GRAD>
__global__ __launch_bounds__(kT) void ce_kernel(void *logits, int64_t ld, const int32_t *targets, float *rowloss, int V, float inv_T) {
  __shared__ float sh[4];
  const int64_t base = (int64_t)blockIdx.x * ld;
  float m = -INFINITY;
  for (int c = threadIdx.x; c < V; c += kT) m = fmaxf(m, El<BF>::ld(logits, base + c));
  m = block_max(m, sh);
  float s = 0.f;
  for (int c = threadIdx.x; c < V; c += kT) s += __expf(El<BF>::ld(logits, base + c) - m);
  s = block_sum(s, sh);
  const float lse = m + logf(s);
  const int tgt = targets[blockIdx.x];
  if (threadIdx.x == 0) rowloss[blockIdx.x] = lse - El<BF>::ld(logits, base + tgt);
  if (!GRAD) return;
  __syncthreads();
  for (int c = threadIdx.x; c < V; c += kT) {
    float p = __expf(El<BF>::ld(logits, base + c) - lse);
    El<BF>::st(logits, base + c, (p - (c == tgt ? 1.f : 0.f)) * inv_T);
  }
  // columns between V and the padded row stride are read (times zero weights) by the next projection
  for (int c = V + threadIdx.x; c < ld; c += kT) El<BF>::st(logits, base + c, 0.f);
}

// row loss from (maximum, sum of exponentials) pairs of its blocks of columns; a wave per row
__global__ __launch_bounds__(kT) void ce_parts_kernel(const f32x2v *parts, int blocks, float *rowloss, int T) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= T) return;
  const f32x2v *p = parts + (int64_t)row * blocks;
  float m = -INFINITY;
  for (int k = lane; k < blocks; k += 64) m = fmaxf(m, p[k].x);
  m = wave_max(m);
  const float ref = m == -INFINITY ? 0.f : m;
  float s = 0.f;
  for (int k = lane; k < blocks; k += 64) s += p[k].y * __expf(p[k].x - ref);
  s = wave_sum(s);
  if (lane == 0) rowloss[row] = m + logf(s) - rowloss[row];
}

__global__ __launch_bounds__(kT) void mean_kernel(const float *v, int64_t n, float scale, float *out) {
  __shared__ float sh[4];
  float part[8] = {};
  for (int64_t i = threadIdx.x; i < n; i += 8 * kT)  // eight loads in flight: 8192 row losses 13 -> 5 us
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t j = i + k * kT;
      const float x = v[j < n ? j : n - 1];
      part[k] += j < n ? x : 0.f;
    }
  const float s = block_sum(((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7])), sh);
  if (threadIdx.x == 0) *out = s * scale;
}

template <int BF>
__global__ __launch_bounds__(kT) void mse_kernel(const float *x, const void *y, float *dx, void *dxb, float *partial, int64_t n, float two_over_n) {
  __shared__ float sh[4];
  float s = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    float d = x[i] - El<BF>::ld(y, i);
    s += d * d;
    float g = d * two_over_n;
    dx[i] = g;
    El<BF>::st(dxb, i, g);
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// ------------------------------------------------------------------------------------------- optimizers
template <int BF>
__global__ __launch_bounds__(kT) void sgd_kernel(void *params, float *master, const float *grads, int64_t n, float lr) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  if (BF) {
    float w = master[i] - lr * grads[i];
    master[i] = w;
    El<BF>::st(params, i, w);
  } else {
    static_cast<float *>(params)[i] -= lr * grads[i];
  }
}

// `first`: the moments count as zero and are not read (a subnet's first step after extraction).
template <int BF>
__global__ __launch_bounds__(kT) void adamw_kernel(void *params, float *master, const float *grads, float *m, float *v, int64_t n, int64_t n_decay,
                                                    float lr, float b1, float b2, float eps, float wd, float inv_bc1, float inv_bc2, int first) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const float g = grads[i];
  const float m0 = first ? 0.f : m[i], v0 = first ? 0.f : v[i];
  const float mi = b1 * m0 + (1.f - b1) * g;
  const float vi = b2 * v0 + (1.f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  float w = BF ? master[i] : static_cast<float *>(params)[i];
  const float decay = i < n_decay ? wd : 0.f;
  w -= lr * ((mi * inv_bc1) / (sqrtf(vi * inv_bc2) + eps) + decay * w);
  if (BF) { master[i] = w; El<BF>::st(params, i, w); }
  else static_cast<float *>(params)[i] = w;
}

__global__ __launch_bounds__(kT) void zero_f32_kernel(float *p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// ------------------------------------------------------------------------------------------- 16-byte paths (bf16)
// Eight bf16 values per thread and access, used when rows are multiples of 8 elements and bases 16-byte aligned.
struct F8 { float v[8]; };
__device__ __forceinline__ F8 unpack8(const u32x4v &u) {
  F8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) { r.v[2 * i] = __uint_as_float(u[i] << 16); r.v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u); }
  return r;
}
__device__ __forceinline__ u32x4v pack8(const F8 &f) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  u32x4v u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f2 p = {f.v[2 * i], f.v[2 * i + 1]};
    u[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(p, b2));  // round to nearest even
  }
  return u;
}

// Cross-entropy of a bf16 row of at most NV * 8 * NT logits held in registers: one read of the row, one write of its gradient where
// that is wanted (GRAD).  Bound by memory; ld8 = row stride / 8; columns between V and the stride are padding and get zeros.
// 512 threads take rows of up to 65536: 8192 x 50257 in 347 us (4.7 TB/s), where the two passes over the row of ce_vec_long_kernel, which
// longer rows still use, take 418.  Without the gradient, which an evaluation has no use for, 4096 x 50257 takes 80 us instead of 212.
// A wave leaves out the vectors that lie beyond the row: 4096 x 515 13.6 us (20.4 if it works on all four), 4096 x 8200 39.5 (60.6 on
// all sixteen), 4096 x 33001 114 (132).
template <int NV, int NT, bool GRAD>
__global__ __launch_bounds__(NT) void ce_vec_kernel(u32x4v *logits, int64_t ld8, const int32_t *targets, float *rowloss, int V, float inv_T) {
  constexpr int NW = NT / 64;
  __shared__ float sh[2][NW];
  u32x4v *row = logits + (int64_t)blockIdx.x * ld8;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mine = (int)ld8 - 64 * wave;  // k NT >= mine: all of the wave's vector k lies beyond the row, and is skipped
  u32x4v x[NV];
  float m = -INFINITY;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int idx = k * NT + threadIdx.x;
    x[k] = u32x4v{0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u};  // -inf: beyond the row
    if (idx < ld8) x[k] = row[idx];
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    if (k * NT < mine) {
      const int left = V - 8 * (k * NT + (int)threadIdx.x);  // logits from this vector on; padding becomes -inf
      if (left < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e >= left) x[k][e >> 1] = e & 1 ? (x[k][e >> 1] & 0xffffu) | 0xff800000u : (x[k][e >> 1] & 0xffff0000u) | 0xff80u;
      }
      const F8 f = unpack8(x[k]);
#pragma unroll
      for (int e = 0; e < 8; ++e) m = fmaxf(m, f.v[e]);
    }
  }
  // (the row stays packed between the passes: unpacked it would take twice the registers and leave half the waves in flight)
#define TW_KEEP_PACKED _Pragma("unroll") for (int k = 0; k < NV; ++k) asm volatile("" : "+v"(x[k]))
  TW_KEEP_PACKED;
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) sh[0][wave] = m;
  __syncthreads();
  m = sh[0][0];
#pragma unroll
  for (int i = 1; i < NW; ++i) m = fmaxf(m, sh[0][i]);
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    if (k * NT < mine) {
      const F8 f = unpack8(x[k]);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += __expf(f.v[e] - m);
    }
  }
  TW_KEEP_PACKED;
#undef TW_KEEP_PACKED
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[1][wave] = s;
  __syncthreads();
  s = sh[1][0];
#pragma unroll
  for (int i = 1; i < NW; ++i) s += sh[1][i];
  const float lse = m + logf(s);
  const int tgt = targets[blockIdx.x];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int idx = k * NT + threadIdx.x;
    if (idx < ld8 && (GRAD || idx == tgt >> 3)) {
      const F8 f = unpack8(x[k]);
      F8 g;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = idx * 8 + e;
        if (c == tgt) rowloss[blockIdx.x] = lse - f.v[e];
        g.v[e] = c < V ? (__expf(f.v[e] - lse) - (c == tgt ? 1.f : 0.f)) * inv_T : 0.f;
      }
      if (GRAD) row[idx] = pack8(g);
    }
  }
}

// The same for fp32 rows of at most NV * 4 * NT logits: bound by memory as well, where ce_kernel reads a row three times, four bytes to a lane and
// load: 1024 x 50257 229 -> 85 us, 4.8 TB/s.
template <int NV, int NT, bool GRAD>
__global__ __launch_bounds__(NT) void ce_vec_f32_kernel(f32x4v *logits, int64_t ld4, const int32_t *targets, float *rowloss, int V, float inv_T) {
  constexpr int NW = NT / 64;
  __shared__ float sh[2][NW];
  f32x4v *row = logits + (int64_t)blockIdx.x * ld4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mine = (int)ld4 - 64 * wave;  // k NT >= mine: all of the wave's vector k lies beyond the row, and is skipped
  f32x4v x[NV];
  float m = -INFINITY;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int idx = k * NT + threadIdx.x;
    x[k] = f32x4v{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (idx < ld4) x[k] = row[idx];
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    if (k * NT < mine) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (4 * (k * NT + (int)threadIdx.x) + e >= V) x[k][e] = -INFINITY;  // padding
        m = fmaxf(m, x[k][e]);
      }
    }
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) sh[0][wave] = m;
  __syncthreads();
  m = sh[0][0];
#pragma unroll
  for (int i = 1; i < NW; ++i) m = fmaxf(m, sh[0][i]);
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    if (k * NT < mine) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s += __expf(x[k][e] - m);
    }
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) sh[1][wave] = s;
  __syncthreads();
  s = sh[1][0];
#pragma unroll
  for (int i = 1; i < NW; ++i) s += sh[1][i];
  const float lse = m + logf(s);
  const int tgt = targets[blockIdx.x];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int idx = k * NT + threadIdx.x;
    if (idx < ld4 && (GRAD || idx == tgt >> 2)) {
      f32x4v g;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 4 * idx + e;
        if (c == tgt) rowloss[blockIdx.x] = lse - x[k][e];
        // columns between V and the row stride are read (times zero weights) by the next projection
        g[e] = c < V ? (__expf(x[k][e] - lse) - (c == tgt ? 1.f : 0.f)) * inv_T : 0.f;
      }
      if (GRAD) row[idx] = g;
    }
  }
}

// The same for rows of any length (row stride a multiple of 8): one vectorised pass keeps a running maximum and a
// sum of exponentials relative to it, a second pass re-reads the row (it is still in the L2) and writes the gradient.
template <bool GRAD>
__global__ __launch_bounds__(kT) void ce_vec_long_kernel(u32x4v *logits, int64_t ld8, const int32_t *targets, float *rowloss, int V, float inv_T) {
  __shared__ float sh[4];
  u32x4v *row = logits + (int64_t)blockIdx.x * ld8;
  float m = -INFINITY, s = 0.f;
  for (int idx = threadIdx.x; idx < ld8; idx += kT) {
    const F8 x = unpack8(row[idx]);
    float mx = m;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (idx * 8 + e < V) mx = fmaxf(mx, x.v[e]);
    if (mx == -INFINITY) continue;  // nothing but padding so far
    float t = s * __expf(m - mx);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (idx * 8 + e < V) t += __expf(x.v[e] - mx);
    m = mx;
    s = t;
  }
  const float M = block_max(m, sh);
  s = block_sum(m == -INFINITY ? 0.f : s * __expf(m - M), sh);
  const float lse = M + logf(s);
  const int tgt = targets[blockIdx.x];
  for (int64_t idx = GRAD ? threadIdx.x : threadIdx.x == 0 && tgt >= 0 ? tgt >> 3 : ld8; idx < ld8; idx += kT) {
    const F8 x = unpack8(row[idx]);
    F8 g;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = (int)idx * 8 + e;
      if (c == tgt) rowloss[blockIdx.x] = lse - x.v[e];
      g.v[e] = c < V ? (__expf(x.v[e] - lse) - (c == tgt ? 1.f : 0.f)) * inv_T : 0.f;
    }
    if (!GRAD) break;
    row[idx] = pack8(g);
  }
}

// a = silu(g) * u on [T, 2F] (gate | up) -> [T, F]; i8 runs over T * F/8
// multiplies the 8 values of columns col0 .. col0 + 7 by the block mask (see act_fwd_kernel)
__device__ __forceinline__ void mask8(F8 &x, const int32_t *keep, int unit, int col0) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
    if (keep[(col0 + e) / unit] < 0) x.v[e] = 0.f;
}

__global__ __launch_bounds__(kT) void swiglu_fwd_vec_kernel(const u32x4v *gu, u32x4v *a, int F8n, int64_t total, const int32_t *keep, int unit) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int64_t t = i / F8n;
  const int c = (int)(i - t * F8n);
  const F8 g = unpack8(gu[t * 2 * F8n + c]), u = unpack8(gu[t * 2 * F8n + F8n + c]);
  F8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o.v[e] = g.v[e] * sigmoidf(g.v[e]) * u.v[e];
  if (keep) mask8(o, keep, unit, 8 * c);
  a[i] = pack8(o);
}

// ungated activations (GELU, ReLU), eight values per thread
// F8n = F / 8 (a row's 8-column groups) where a mask is given, so that a thread knows its columns
__global__ __launch_bounds__(kT) void act_fwd_vec_kernel(int act, const u32x4v *u, u32x4v *a, int64_t total, const int32_t *keep, int unit, int F8n) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const F8 x = unpack8(u[i]);
  F8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o.v[e] = act_value<false>(act, x.v[e]);
  if (keep) mask8(o, keep, unit, 8 * (int)(i % F8n));
  a[i] = pack8(o);
}

__global__ __launch_bounds__(kT) void act_bwd_vec_kernel(int act, const u32x4v *u, const u32x4v *da, u32x4v *du, int64_t total, const int32_t *keep, int unit,
                                                          int F8n) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const F8 x = unpack8(u[i]);
  F8 d = unpack8(da[i]);
  if (keep) mask8(d, keep, unit, 8 * (int)(i % F8n));
  F8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o.v[e] = d.v[e] * (act == TWIST_ACT_RELU ? (x.v[e] > 0.f ? 1.f : 0.f) : gelu_tanh_grad<false>(x.v[e]));
  du[i] = pack8(o);
}

// The same, and the column sums of du over chunks of kChunkRows rows (the up projection's bias gradient), which a kernel of its own would read
// du again for.  A workgroup owns 64 (chunk, 8 columns) pairs, a wave a quarter of their rows: 8192 x 768
// 8.7 + 4.9 us -> 10.6, bound by the arithmetic of the gradient as much as by its 38 MB.
__global__ __launch_bounds__(kT) void act_bwd_sum_kernel(int act, const u32x4v *u, const u32x4v *da, u32x4v *du, float *partial, int T, int n8, int64_t pairs,
                                                          const int32_t *keep, int unit) {
  constexpr int R = kChunkRows / 4;
  __shared__ f32x4v sh[3][2][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const bool mine = i < pairs;
  const int chunk = mine ? (int)(i / n8) : 0, v = mine ? (int)(i - (int64_t)chunk * n8) : 0, r0 = chunk * kChunkRows + R * wave;
  u32x4v x[R], y[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t at = (int64_t)min(r0 + r, T - 1) * n8 + v;
    x[r] = u[at];
    y[r] = da[at];
  }
  f32x4v lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const F8 a = unpack8(x[r]);
    F8 d = unpack8(y[r]), o;
    if (keep) mask8(d, keep, unit, 8 * v);
#pragma unroll
    for (int e = 0; e < 8; ++e) o.v[e] = d.v[e] * (act == TWIST_ACT_RELU ? (a.v[e] > 0.f ? 1.f : 0.f) : gelu_tanh_grad<false>(a.v[e]));
    const u32x4v p = pack8(o);
    if (mine && r0 + r < T) {
      du[(int64_t)(r0 + r) * n8 + v] = p;
      const F8 s = unpack8(p);  // as stored
#pragma unroll
      for (int e = 0; e < 4; ++e) { lo[e] += s.v[e]; hi[e] += s.v[4 + e]; }
    }
  }
  if (wave) { sh[wave - 1][0][lane] = lo; sh[wave - 1][1][lane] = hi; }
  __syncthreads();
  if (wave || !mine) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) { lo += sh[k][0][lane]; hi += sh[k][1][lane]; }
  f32x4v *o = reinterpret_cast<f32x4v *>(partial) + 2 * i;
  o[0] = lo;
  o[1] = hi;
}

__global__ __launch_bounds__(kT) void swiglu_bwd_vec_kernel(const u32x4v *gu, const u32x4v *da, u32x4v *dgu, int F8n, int64_t total, const int32_t *keep,
                                                             int unit) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int64_t t = i / F8n;
  const int c = (int)(i - t * F8n);
  const F8 g = unpack8(gu[t * 2 * F8n + c]), u = unpack8(gu[t * 2 * F8n + F8n + c]);
  F8 d = unpack8(da[i]);
  if (keep) mask8(d, keep, unit, 8 * c);
  F8 dg, du;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float sg = sigmoidf(g.v[e]);
    du.v[e] = d.v[e] * g.v[e] * sg;
    dg.v[e] = d.v[e] * u.v[e] * (sg + g.v[e] * sg * (1.f - sg));
  }
  dgu[t * 2 * F8n + c] = pack8(dg);
  dgu[t * 2 * F8n + F8n + c] = pack8(du);
}

// rotation of the q and k heads of a fused [T, 3 Hs dh] buffer; i runs over T * 2Hs * (dh/16): 8 pairs per thread
__global__ __launch_bounds__(kT) void rope_vec_kernel(u32x4v *qkv, const float *tab, int N, int Hs, int dh, float sign, int64_t total) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int half = dh / 2, h8 = half / 8;
  const int f8 = (int)(i % h8);
  const int64_t r = i / h8;
  const int head = (int)(r % (2 * Hs));
  const int64_t t = r / (2 * Hs);
  const int pos = (int)(t % N);
  const int64_t base = (t * (3 * (int64_t)Hs * dh) + (int64_t)head * dh) / 8 + f8;
  const F8 a = unpack8(qkv[base]), b = unpack8(qkv[base + h8]);
  const f32x4v *cs = reinterpret_cast<const f32x4v *>(tab + 2 * ((int64_t)pos * half + 8 * f8));  // (cos, sin) pairs
  F8 oa, ob;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const f32x4v w = cs[e];
    oa.v[2 * e] = a.v[2 * e] * w[0] - b.v[2 * e] * (sign * w[1]);
    ob.v[2 * e] = b.v[2 * e] * w[0] + a.v[2 * e] * (sign * w[1]);
    oa.v[2 * e + 1] = a.v[2 * e + 1] * w[2] - b.v[2 * e + 1] * (sign * w[3]);
    ob.v[2 * e + 1] = b.v[2 * e + 1] * w[2] + a.v[2 * e + 1] * (sign * w[3]);
  }
  qkv[base] = pack8(oa);
  qkv[base + h8] = pack8(ob);
}

// norm forward for rows of D <= NV * 256 elements, D a multiple of 4: a wave per row, the row held in registers (vectors beyond D as in the
// backward kernel).  fp32 8192 x 2048 32 -> 20 us, bf16 4000 x 1304 16 -> 8.7 (one value a lane and three passes over the row
// before); FULL: D = NV * 256.
template <int BF, int RMS, int NV, bool FULL>
__global__ __launch_bounds__(kT) void norm_fwd_vec_kernel(const float *x, const void *w, const void *b, void *y, float *stats, int T, int Dn, float eps) {
  const int D = FULL ? NV * 256 : Dn;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, d4 = D >> 2;
  if (row >= T) return;
  const int64_t rv = (int64_t)row * d4;
  auto on = [&](int k) { return FULL || lane + 64 * k < d4; };
  auto at = [&](int k) { return FULL ? lane + 64 * k : min(lane + 64 * k, d4 - 1); };
  f32x4v xv[NV], wv[NV], bv[NV];
  auto gains = [&](int k) {
    const int v = at(k);
    wv[k] = ld4<BF>(w, v);
    bv[k] = b ? ld4<BF>(b, v) : f32x4v{0.f, 0.f, 0.f, 0.f};
  };
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    xv[k] = reinterpret_cast<const f32x4v *>(x)[rv + at(k)];
    if (NV <= 4) gains(k);  // (longer rows: in time enough, and in fewer registers, behind the sums)
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) s += on(k) ? xv[k][0] + xv[k][1] + xv[k][2] + xv[k][3] : 0.f;
  const float mean = RMS ? 0.f : wave_sum(s) / D;
  float s2 = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    xv[k] -= mean;
    s2 += on(k) ? xv[k][0] * xv[k][0] + xv[k][1] * xv[k][1] + xv[k][2] * xv[k][2] + xv[k][3] * xv[k][3] : 0.f;
  }
  const float rstd = 1.0f / sqrtf(wave_sum(s2) / D + eps);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    if (NV > 4) gains(k);
    if (!on(k)) continue;
    f32x4v o = xv[k] * rstd * wv[k];
    if (b) o += bv[k];
    st4<BF>(y, rv + lane + 64 * k, o);
  }
  if (lane == 0) { stats[2 * row] = mean; stats[2 * row + 1] = rstd; }
}

inline dim3 grid1(int64_t n) { return dim3((unsigned)((n + kT - 1) / kT)); }

}  // namespace

#define LAUNCH_BF(kern, bf, grid, block, ...)                                             \
  do {                                                                                    \
    if (bf) hipLaunchKernelGGL((kern<1>), grid, block, 0, ctx->stream, __VA_ARGS__);      \
    else hipLaunchKernelGGL((kern<0>), grid, block, 0, ctx->stream, __VA_ARGS__);         \
    TW_HIP(ctx, hipGetLastError());                                                       \
  } while (0)

#define LAUNCH_BF2(kern, bf, flag, grid, block, ...)                                                  \
  do {                                                                                                \
    if (bf && flag) hipLaunchKernelGGL((kern<1, 1>), grid, block, 0, ctx->stream, __VA_ARGS__);       \
    else if (bf) hipLaunchKernelGGL((kern<1, 0>), grid, block, 0, ctx->stream, __VA_ARGS__);          \
    else if (flag) hipLaunchKernelGGL((kern<0, 1>), grid, block, 0, ctx->stream, __VA_ARGS__);        \
    else hipLaunchKernelGGL((kern<0, 0>), grid, block, 0, ctx->stream, __VA_ARGS__);                  \
    TW_HIP(ctx, hipGetLastError());                                                                   \
  } while (0)

twist_status twist_zero_f32(twist_ctx *ctx, float *p, int64_t n) {
  if (n <= 0) return TWIST_OK;
  hipLaunchKernelGGL(zero_f32_kernel, grid1(n), dim3(kT), 0, ctx->stream, p, n);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

static bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

twist_status twist_embed_fwd(twist_ctx *ctx, int bf16, const int32_t *tok, const void *E, const void *P, float *x, int B, int N, int D, int) {
  const int64_t T = (int64_t)B * N;
  const dim3 grid((unsigned)((T + 3) / 4)), block(kT);
  const bool vec = D % 4 == 0 && al16(E) && al16(P) && al16(x);
#define TW_EMBED(BF, VEC) hipLaunchKernelGGL((embed_fwd_kernel<BF, VEC>), grid, block, 0, ctx->stream, tok, E, P, x, N, D, T)
  if (bf16) { if (vec) TW_EMBED(1, true); else TW_EMBED(1, false); }
  else { if (vec) TW_EMBED(0, true); else TW_EMBED(0, false); }
#undef TW_EMBED
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_embed_bwd(twist_ctx *ctx, const int32_t *tok, const float *dx, float *d_tok, float *d_pos, int B, int N, int D) {
  const int64_t T = (int64_t)B * N;
  hipLaunchKernelGGL(embed_bwd_tok_kernel, dim3((unsigned)((T + 3) / 4)), dim3(kT), 0, ctx->stream, tok, dx, d_tok, D, T);
  TW_HIP(ctx, hipGetLastError());
  if (d_pos) {
    hipLaunchKernelGGL(embed_bwd_pos_kernel, grid1((int64_t)N * D), dim3(kT), 0, ctx->stream, dx, d_pos, B, N, D);
    TW_HIP(ctx, hipGetLastError());
  }
  return TWIST_OK;
}

twist_status twist_cast_in(twist_ctx *ctx, int bf16, const void *src, float *dst, int64_t n) {
  LAUNCH_BF(cast_in_kernel, bf16, grid1(n), dim3(kT), src, dst, n);
  return TWIST_OK;
}

// vectors of 256 columns that the register-held norm kernels are built for, enough for rows of D (0: too long, or not a multiple of 4)
static int norm_vectors(int D) {
  if (D % 4 || D > 4096) return 0;
  const int n = (D + 255) / 256;
  return n <= 4 ? n : n <= 6 ? 6 : n <= 8 ? 8 : n <= 12 ? 12 : 16;
}

twist_status twist_norm_fwd(twist_ctx *ctx, int bf16, int rms, const float *x, const void *w, const void *b, void *y, float *stats, int T, int D, float eps) {
  const int nv = norm_vectors(D);
  if (nv && al16(x) && al16(w) && al16(y) && (!b || al16(b))) {
#define TW_NORM_FWD(BF, RMS, NV)                                                                                                                                          \
  do {                                                                                                                                                                   \
    if (D == NV * 256) hipLaunchKernelGGL((norm_fwd_vec_kernel<BF, RMS, NV, true>), dim3((T + 3) / 4), dim3(kT), 0, ctx->stream, x, w, b, y, stats, T, D, eps);            \
    else hipLaunchKernelGGL((norm_fwd_vec_kernel<BF, RMS, NV, false>), dim3((T + 3) / 4), dim3(kT), 0, ctx->stream, x, w, b, y, stats, T, D, eps);                        \
  } while (0)
#define TW_NORM_FWD4(NV)                     \
  do {                                       \
    if (bf16 && rms) TW_NORM_FWD(1, 1, NV);  \
    else if (bf16) TW_NORM_FWD(1, 0, NV);    \
    else if (rms) TW_NORM_FWD(0, 1, NV);     \
    else TW_NORM_FWD(0, 0, NV);              \
  } while (0)
    switch (nv) {
      case 1: TW_NORM_FWD4(1); break;
      case 2: TW_NORM_FWD4(2); break;
      case 3: TW_NORM_FWD4(3); break;
      case 4: TW_NORM_FWD4(4); break;
      case 6: TW_NORM_FWD4(6); break;
      case 8: TW_NORM_FWD4(8); break;
      case 12: TW_NORM_FWD4(12); break;
      default: TW_NORM_FWD4(16); break;
    }
#undef TW_NORM_FWD4
#undef TW_NORM_FWD
    TW_HIP(ctx, hipGetLastError());
    return TWIST_OK;
  }
  LAUNCH_BF2(norm_fwd_kernel, bf16, rms, dim3((T + 3) / 4), dim3(kT), x, w, b, y, stats, T, D, eps);
  return TWIST_OK;
}

static int n_chunks(int T) { return (T + kChunkRows - 1) / kChunkRows; }
size_t twist_norm_partial_floats(int T, int D) { return (size_t)n_chunks(T) * 2 * D; }
size_t twist_colsum_partial_floats(int T, int n) { return (size_t)n_chunks(T) * n; }

twist_status twist_norm_bwd(twist_ctx *ctx, int bf16, int rms, const void *dy, const float *x, const void *w, const float *stats, float *dx,
                            int accumulate, void *dxb, float *dw, float *db, float *partial, int T, int D, bool defer_reduce, float *csum) {
  const int nc = n_chunks(T);
  const int nv = norm_vectors(D);
  const bool cs_ok = csum && al16(csum) && dxb;
  if (nv && al16(dy) && al16(x) && al16(w) && al16(dx) && al16(partial) && (!dxb || al16(dxb))) {
    float *fcs = cs_ok && (nv <= 4 || nv >= 12) ? csum : nullptr;  // rows of 6 and 8 vectors: the third set of sums costs the kernel half its waves
    const bool few = nc < 256;
#define TW_NORM_BWD2(BF, RMS, NV, CS, W, FULL) \
  hipLaunchKernelGGL((norm_bwd_fused_kernel<BF, RMS, NV, CS, W, FULL>), dim3(nc), dim3(64 * (W)), 0, ctx->stream, dy, x, w, stats, dx, accumulate, dxb, partial, fcs, T, D)
#define TW_NORM_BWD(BF, RMS, NV, CS, W)                              \
  do {                                                               \
    if (D == NV * 256) TW_NORM_BWD2(BF, RMS, NV, CS, W, true);       \
    else TW_NORM_BWD2(BF, RMS, NV, CS, W, false);                    \
  } while (0)
#define TW_NORM_SHORT(BF, RMS, NV)                          \
  do {                                                      \
    if (fcs && few) TW_NORM_BWD(BF, RMS, NV, true, 8);      \
    else if (fcs) TW_NORM_BWD(BF, RMS, NV, true, 4);        \
    else if (few) TW_NORM_BWD(BF, RMS, NV, false, 8);       \
    else TW_NORM_BWD(BF, RMS, NV, false, 4);                \
  } while (0)
#define TW_NORM_LONG(BF, RMS, NV) TW_NORM_BWD(BF, RMS, NV, false, 4)
#define TW_NORM_WIDE(BF, RMS, NV)                                                                                                                             \
  do {                                                                                                                                                         \
    if (fcs) hipLaunchKernelGGL((norm_bwd_wide_kernel<BF, RMS, NV, true>), dim3(nc), dim3(kT), 0, ctx->stream, dy, x, w, stats, dx, accumulate, dxb, partial, fcs, T, D);  \
    else hipLaunchKernelGGL((norm_bwd_wide_kernel<BF, RMS, NV, false>), dim3(nc), dim3(kT), 0, ctx->stream, dy, x, w, stats, dx, accumulate, dxb, partial, fcs, T, D);      \
  } while (0)
#define TW_NORM_FUSED(KIND, NV)                \
  do {                                         \
    if (bf16 && rms) KIND(1, 1, NV);           \
    else if (bf16) KIND(1, 0, NV);             \
    else if (rms) KIND(0, 1, NV);              \
    else KIND(0, 0, NV);                       \
  } while (0)
    switch (nv) {
      case 1: TW_NORM_FUSED(TW_NORM_SHORT, 1); break;
      case 2: TW_NORM_FUSED(TW_NORM_SHORT, 2); break;
      case 3: TW_NORM_FUSED(TW_NORM_SHORT, 3); break;
      case 4: TW_NORM_FUSED(TW_NORM_SHORT, 4); break;
      case 6: TW_NORM_FUSED(TW_NORM_LONG, 6); break;
      case 8: TW_NORM_FUSED(TW_NORM_LONG, 8); break;
      case 12: TW_NORM_FUSED(TW_NORM_WIDE, 3); break;
      default: TW_NORM_FUSED(TW_NORM_WIDE, 4); break;
    }
#undef TW_NORM_WIDE
#undef TW_NORM_FUSED
#undef TW_NORM_LONG
#undef TW_NORM_SHORT
#undef TW_NORM_BWD
#undef TW_NORM_BWD2
    TW_HIP(ctx, hipGetLastError());
    if (csum && !fcs) TW_TRY(twist_colsum(ctx, bf16, dxb, D, 1.f, nullptr, csum, T, D, true));
    if (defer_reduce) return TWIST_OK;
    hipLaunchKernelGGL(reduce_partial_kernel, dim3((D + 15) / 16), dim3(kT), 0, ctx->stream, partial, (int64_t)2 * D, nc, 1.f, dw, D);
    if (db) hipLaunchKernelGGL(reduce_partial_kernel, dim3((D + 15) / 16), dim3(kT), 0, ctx->stream, partial + D, (int64_t)2 * D, nc, 1.f, db, D);
    TW_HIP(ctx, hipGetLastError());
    return TWIST_OK;
  }
  // general shapes: parameter gradients first (they read dy and x, which the dx pass leaves untouched)
  LAUNCH_BF(norm_bwd_dw_kernel, bf16, dim3((D + 63) / 64, nc), dim3(64), dy, x, stats, partial, T, D);
  if (!defer_reduce) hipLaunchKernelGGL(reduce_partial_kernel, dim3((D + 15) / 16), dim3(kT), 0, ctx->stream, partial, (int64_t)2 * D, nc, 1.f, dw, D);
  TW_HIP(ctx, hipGetLastError());
  if (db && !defer_reduce) {
    hipLaunchKernelGGL(reduce_partial_kernel, dim3((D + 15) / 16), dim3(kT), 0, ctx->stream, partial + D, (int64_t)2 * D, nc, 1.f, db, D);
    TW_HIP(ctx, hipGetLastError());
  }
  LAUNCH_BF2(norm_bwd_dx_kernel, bf16, rms, dim3((T + 3) / 4), dim3(kT), dy, x, w, stats, dx, accumulate, dxb, T, D);
  if (csum) return twist_colsum(ctx, bf16, dxb, D, 1.f, nullptr, csum, T, D, true);
  return TWIST_OK;
}

twist_status twist_col_reduce_batch(twist_ctx *ctx, const ColReduce *items, int n_items, int T) {
  const int nc = n_chunks(T);
  for (int i0 = 0; i0 < n_items; i0 += kReduceBatch) {
    ColReduceArgs a;
    const int m = std::min(kReduceBatch, n_items - i0);
    int widest = 1;
    bool vec = true;
    for (int i = 0; i < m; ++i) {
      const ColReduce &it = a.item[i] = items[i0 + i];
      widest = std::max(widest, it.n);
      vec = vec && it.n % 4 == 0 && it.stride % 4 == 0 && al16(it.partial);
    }
    if (vec) hipLaunchKernelGGL(reduce_partial_batch_vec_kernel, dim3((widest + 63) / 64, m), dim3(kT), 0, ctx->stream, a, nc);
    else hipLaunchKernelGGL(reduce_partial_batch_kernel, dim3((widest + 15) / 16, m), dim3(kT), 0, ctx->stream, a, nc);
    TW_HIP(ctx, hipGetLastError());
  }
  return TWIST_OK;
}

twist_status twist_colsum(twist_ctx *ctx, int bf16, const void *src, int64_t ld, float alpha, float *out, float *partial, int T, int n,
                          bool defer_reduce) {
  const int nc = n_chunks(T), per = bf16 ? 8 : 4;
  if (n % per == 0 && ld % per == 0 && al16(src) && al16(partial)) {
    const int64_t total = (int64_t)(n / per) * nc;
    LAUNCH_BF(colsum_vec_kernel, bf16, dim3((unsigned)((total + kT - 1) / kT)), dim3(kT), src, ld, partial, T, n, n / per, total);
  } else
    LAUNCH_BF(colsum_kernel, bf16, dim3((n + 63) / 64, nc), dim3(64), src, ld, partial, T, n);
  if (defer_reduce) return TWIST_OK;
  hipLaunchKernelGGL(reduce_partial_kernel, dim3((n + 15) / 16), dim3(kT), 0, ctx->stream, partial, (int64_t)n, nc, alpha, out, n);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

// rotary table lives at the start of `qkv`-independent scratch handed in by the caller through twist_rope_table
twist_status twist_rope_table(twist_ctx *ctx, float *tab, int N, int dh, float theta) {
  const int half = dh / 2;
  hipLaunchKernelGGL(rope_table_kernel, grid1((int64_t)N * half), dim3(kT), 0, ctx->stream, tab, N, half, dh, theta);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_rope_apply(twist_ctx *ctx, int bf16, void *qkv, const float *tab, int B, int N, int Hs, int dh, float sign) {
  if (bf16 && dh % 16 == 0 && al16(qkv) && al16(tab)) {
    const int64_t total8 = (int64_t)B * N * 2 * Hs * (dh / 16);
    hipLaunchKernelGGL(rope_vec_kernel, grid1(total8), dim3(kT), 0, ctx->stream, static_cast<u32x4v *>(qkv), tab, N, Hs, dh, sign, total8);
    TW_HIP(ctx, hipGetLastError());
    return TWIST_OK;
  }
  const int64_t total = (int64_t)B * N * 2 * Hs * (dh / 2);
  LAUNCH_BF(rope_kernel, bf16, grid1(total), dim3(kT), qkv, tab, N, Hs, dh, sign, total);
  return TWIST_OK;
}

twist_status twist_act_fwd(twist_ctx *ctx, int bf16, int act, const void *gu, void *a, int T, int F, const int32_t *keep, int unit) {
  const int64_t total = (int64_t)T * F;
  if (bf16 && act == TWIST_ACT_SWIGLU && F % 8 == 0 && al16(gu) && al16(a)) {
    hipLaunchKernelGGL(swiglu_fwd_vec_kernel, grid1(total / 8), dim3(kT), 0, ctx->stream, static_cast<const u32x4v *>(gu), static_cast<u32x4v *>(a), F / 8, total / 8,
                       keep, unit);
    TW_HIP(ctx, hipGetLastError());
    return TWIST_OK;
  }
  if (bf16 && act != TWIST_ACT_SWIGLU && (keep ? F % 8 == 0 : total % 8 == 0) && al16(gu) && al16(a)) {
    hipLaunchKernelGGL(act_fwd_vec_kernel, grid1(total / 8), dim3(kT), 0, ctx->stream, act, static_cast<const u32x4v *>(gu), static_cast<u32x4v *>(a), total / 8,
                       keep, unit, F / 8);
    TW_HIP(ctx, hipGetLastError());
    return TWIST_OK;
  }
  LAUNCH_BF(act_fwd_kernel, bf16, grid1(total), dim3(kT), act, gu, a, F, total, keep, unit);
  return TWIST_OK;
}

twist_status twist_act_bwd(twist_ctx *ctx, int bf16, int act, const void *gu, const void *da, void *dgu, int T, int F, const int32_t *keep, int unit,
                           float *sums) {
  const int64_t total = (int64_t)T * F;
  const bool vec = bf16 && al16(gu) && al16(da) && al16(dgu);
  if (vec && sums && act != TWIST_ACT_SWIGLU && F % 8 == 0 && total > 0 && al16(sums)) {
    const int64_t pairs = (int64_t)n_chunks(T) * (F / 8);
    hipLaunchKernelGGL(act_bwd_sum_kernel, dim3((unsigned)((pairs + 63) / 64)), dim3(kT), 0, ctx->stream, act, static_cast<const u32x4v *>(gu),
                       static_cast<const u32x4v *>(da), static_cast<u32x4v *>(dgu), sums, T, F / 8, pairs, keep, unit);
    TW_HIP(ctx, hipGetLastError());
    return TWIST_OK;
  }
  if (vec && act == TWIST_ACT_SWIGLU && F % 8 == 0) {
    hipLaunchKernelGGL(swiglu_bwd_vec_kernel, grid1(total / 8), dim3(kT), 0, ctx->stream, static_cast<const u32x4v *>(gu), static_cast<const u32x4v *>(da),
                       static_cast<u32x4v *>(dgu), F / 8, total / 8, keep, unit);
    TW_HIP(ctx, hipGetLastError());
  } else if (vec && act != TWIST_ACT_SWIGLU && (keep ? F % 8 == 0 : total % 8 == 0)) {
    hipLaunchKernelGGL(act_bwd_vec_kernel, grid1(total / 8), dim3(kT), 0, ctx->stream, act, static_cast<const u32x4v *>(gu), static_cast<const u32x4v *>(da),
                       static_cast<u32x4v *>(dgu), total / 8, keep, unit, F / 8);
    TW_HIP(ctx, hipGetLastError());
  } else {
    LAUNCH_BF(act_bwd_kernel, bf16, grid1(total), dim3(kT), act, gu, da, dgu, F, total, keep, unit);
  }
  const int n = act == TWIST_ACT_SWIGLU ? 2 * F : F;
  return sums ? twist_colsum(ctx, bf16, dgu, n, 1.f, nullptr, sums, T, n, true) : TWIST_OK;
}

twist_status twist_ce_fwd_bwd(twist_ctx *ctx, int bf16, void *logits, int64_t ld, const int32_t *targets, float *rowloss, float *loss, int T, int V, bool grad) {
  const float inv_T = 1.f / (float)T;
#define TW_CE(KERNEL, GRAD, THREADS, ...) hipLaunchKernelGGL((KERNEL<__VA_ARGS__ GRAD>), dim3(T), dim3(THREADS), 0, ctx->stream, lv, LD, targets, rowloss, V, inv_T)
#define TW_CE2(KERNEL, THREADS, ...)                        \
  do {                                                      \
    if (grad) TW_CE(KERNEL, true, THREADS, __VA_ARGS__);    \
    else TW_CE(KERNEL, false, THREADS, __VA_ARGS__);        \
  } while (0)
  if (bf16 && ld % 8 == 0 && al16(logits)) {
    u32x4v *lv = static_cast<u32x4v *>(logits);
    const int64_t LD = ld / 8;
    if (ld <= 4 * 2048) TW_CE2(ce_vec_kernel, kT, 4, kT,);
    else if (ld <= 16 * 2048) TW_CE2(ce_vec_kernel, kT, 16, kT,);
    else if (ld <= 16 * 4096) TW_CE2(ce_vec_kernel, 512, 16, 512,);
    else TW_CE2(ce_vec_long_kernel, kT, );
  } else if (!bf16 && ld % 4 == 0 && ld <= 65536 && al16(logits)) {
    f32x4v *lv = static_cast<f32x4v *>(logits);
    const int64_t LD = ld / 4;
    if (ld <= 4 * 1024) TW_CE2(ce_vec_f32_kernel, kT, 4, kT,);
    else if (ld <= 16 * 1024) TW_CE2(ce_vec_f32_kernel, kT, 16, kT,);
    else if (ld <= 16 * 2048) TW_CE2(ce_vec_f32_kernel, 512, 16, 512,);
    else TW_CE2(ce_vec_f32_kernel, 1024, 16, 1024,);
  } else {
    void *lv = logits;
    const int64_t LD = ld;
    if (bf16) TW_CE2(ce_kernel, kT, 1,);
    else TW_CE2(ce_kernel, kT, 0,);
  }
#undef TW_CE2
#undef TW_CE
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(kT), 0, ctx->stream, rowloss, (int64_t)T, inv_T, loss);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_ce_parts(twist_ctx *ctx, const float *parts, int blocks, float *rowloss, float *loss, int T) {
  hipLaunchKernelGGL(ce_parts_kernel, dim3((T + 3) / 4), dim3(kT), 0, ctx->stream, reinterpret_cast<const f32x2v *>(parts), blocks, rowloss, T);
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(kT), 0, ctx->stream, rowloss, (int64_t)T, 1.f / (float)T, loss);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_mse_fwd_bwd(twist_ctx *ctx, int bf16, const float *x, const void *y, float *dx, void *dxb, float *partial, float *loss, int64_t n) {
  const int blocks = (int)std::min<int64_t>((n + kT - 1) / kT, 1024);
  LAUNCH_BF(mse_kernel, bf16, dim3(blocks), dim3(kT), x, y, dx, dxb, partial, n, 2.f / (float)n);
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(kT), 0, ctx->stream, partial, (int64_t)blocks, 1.f / (float)n, loss);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_sgd(twist_ctx *ctx, int bf16, void *params, float *master, const float *grads, int64_t n, float lr) {
  LAUNCH_BF(sgd_kernel, bf16, grid1(n), dim3(kT), params, master, grads, n, lr);
  return TWIST_OK;
}

twist_status twist_adamw(twist_ctx *ctx, int bf16, void *params, float *master, const float *grads, float *m, float *v, int64_t n, int64_t n_decay,
                         float lr, float b1, float b2, float eps, float wd, int64_t step) {
  const double bc1 = 1.0 - pow((double)b1, (double)step), bc2 = 1.0 - pow((double)b2, (double)step);
  LAUNCH_BF(adamw_kernel, bf16, grid1(n), dim3(kT), params, master, grads, m, v, n, n_decay, lr, b1, b2, eps, wd, (float)(1.0 / bc1), (float)(1.0 / bc2), step == 1 ? 1 : 0);
  return TWIST_OK;
}
