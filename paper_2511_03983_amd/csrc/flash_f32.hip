// Tiled causal attention in fp32 arithmetic on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32), forward and backward,
// d_head a multiple of 4 up to 128, any N: for fp32 models, and (BF) for the bf16 models whose heads are not 32, 64 or 128 wide or whose batch
// element exceeds 2 GiB (flash64.hip): operands and results are bf16 there, probabilities and score gradients stay fp32.
//
// A workgroup owns 32 query rows (forward, dQ) or 32 key rows (dK / dV) of one head; its four or eight (NW) waves share out the tiles of 32 keys
// (or queries) that those rows see, wave w taking tiles w, w + NW, ..., each with accumulators of its own, and the results are
// added in wave order through LDS at the end.  That gives N / 32 workgroups per head, each a quarter or less as long as one wave would be:
// these models are small, and what bounds the kernels is the chain of dependent steps and how many waves there are, then the
// matrix pipes (64 cycles per instruction).  Operands go from global memory to registers: waves share no tile, and a head's keys
// and values stay in the L2.
// As in the bf16 kernels scores are formed transposed (a lane owns a query, or a key in the dK / dV kernel), and a score tile is
// the B operand of the next product as it stands: MFMA number r contracts the rows 8 (r / 4) + 4 g + r % 4 (g = lane / 32), which
// is where accumulator register r sits.  Along d_head, MFMA 4 u + e contracts columns 8 u + 4 g + e: one 16-byte load per lane
// feeds four instructions.
// Rounding (fp32 models; bf16 results are rounded a thousand times coarser): a score is added up in four chains and an exponent is
// formed from the difference of a score and its reference, so that what is rounded is that and not the score, which may be large.
// 2 x 200 tokens, 3 heads of 128, scores of about +-30, error of the output: 10.6e-7 with one chain and score * scale - reference,
// 4.1e-7 like this, 3.5e-7 in the plain kernels, which add pairwise; 2 x 512 tokens, 6 heads of 64, normal operands: 2.3e-7, 1.6e-7
// and 2.5e-7, for 2.5 us of 80 forward and backward.
// delta_i = dO_i . O_i from the fp32 output.  Rows beyond N are clamped when read and not stored; keys beyond N come after
// every query, and queries beyond N get probability zero.  An infinity or a NaN reaches what depends on it and nothing else: no
// query sees a later key's, no key an earlier query's (add_tile).  That costs nothing that can be measured
// (forward and backward of the first shape below: 80.3 us before, 78.6 since).
//
// Measured (forward / dQ / dK dV) on 2 x 512 tokens, 6 heads of 64: 20 / 29 / 36 us against 423 / 905 / 427 us of the plain kernels
// (a wave per row, a wave reduction per score), and closer to exact arithmetic where a value bias cancels (query / key gradients 1.3e-5
// against 3.7e-5).
#include "nn.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32((a), (b), (c), 0, 0, 0)

// element type of the operands and results
template <int BF> struct El { using T = float; };
template <> struct El<1> { using T = uint16_t; };
__device__ __forceinline__ float get(const float *p) { return *p; }
__device__ __forceinline__ float get(const uint16_t *p) { return __uint_as_float((uint32_t)*p << 16); }
__device__ __forceinline__ f32x4 get4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ f32x4 get4(const uint16_t *p) {
  const u32x2 u = *reinterpret_cast<const u32x2 *>(p);
  return f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
}
__device__ __forceinline__ void put4(float *p, const f32x4 &v) { *reinterpret_cast<f32x4 *>(p) = v; }
__device__ __forceinline__ void put4(uint16_t *p, const f32x4 &v) {  // round to nearest even
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 a = {v[0], v[1]}, b = {v[2], v[3]};
  *reinterpret_cast<u32x2 *>(p) = u32x2{__builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf16x2)), __builtin_bit_cast(uint32_t, __builtin_convertvector(b, bf16x2))};
}

// one row's values for the contraction along d_head: group u holds columns 8 u + 4 g .. + 3 (zeros beyond dh)
template <int DH, class T>
__device__ __forceinline__ void load_row(f32x4 (&f)[DH / 8], const T *row, int dh, int g) {
#pragma unroll
  for (int u = 0; u < DH / 8; ++u) {
    const int k = 8 * u + 4 * g;
    f[u] = k < dh ? get4(row + k) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
}
// chains of a score: the same in all kernels, so that the rounding of a score is the same where its probability is formed again
template <int BF> constexpr int kChains = BF ? 1 : 4;
// 32 x 32 tile of A B^T along d_head, summed in CH chains: `a` = this lane's row of A, `b` = this lane's column
template <int DH, int CH>
__device__ __forceinline__ f32x16 dot_tile(const f32x4 (&a)[DH / 8], const f32x4 (&b)[DH / 8]) {
  f32x16 s[CH];
#pragma unroll
  for (int h = 0; h < CH; ++h)
#pragma unroll
    for (int r = 0; r < 16; ++r) s[h][r] = 0.f;
#pragma unroll
  for (int u = 0; u < DH / 8; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e % CH] = MFMA(a[u][e], b[u][e], s[e % CH]);
  return CH == 4 ? (s[0] + s[1 % CH]) + (s[2 % CH] + s[3 % CH]) : CH == 2 ? s[0] + s[1 % CH] : s[0];
}
// the same with this lane's column in LDS (its group u at b + 8 u)
template <int DH, int CH>
__device__ __forceinline__ f32x16 dot_tile(const f32x4 (&a)[DH / 8], const float *b) {
  f32x4 f[DH / 8];
#pragma unroll
  for (int u = 0; u < DH / 8; ++u) f[u] = get4(b + 8 * u);
  return dot_tile<DH, CH>(a, f);
}
// acc[i] += X^T[32 i ..][rows] w[rows][column]: X rows row0 .. row0 + 31 (those beyond N are taken as zero), w in accumulator layout.
// `diag`: the tile lies on the diagonal, where a column does not see every row.  Hidden entries have weight zero, but zero times an
// infinity or a NaN is a NaN, and it must not reach a column that never reads that row: such values are left out here, and if
// there was one the weights are kept in `kept` (32 x 32 floats of LDS) and add_left_out() adds what the columns do see of them.
template <int DH, class T>
__device__ __forceinline__ bool add_tile(f32x16 (&acc)[DH / 32], const T *x, int64_t ld, int row0, int N, int dh, const f32x16 &w, int c, int g, bool diag, float *kept) {
  bool odd = false;
#pragma unroll
  for (int i = 0; i < DH / 32; ++i) {
    if (32 * i >= dh) break;
    const int col = min(32 * i + c, dh - 1);  // columns beyond dh give rows of the result that are not stored
    float v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = get(x + (int64_t)min(row0 + 8 * (r >> 2) + 4 * g + (r & 3), N - 1) * ld + col);
    if (row0 + 32 > N) {
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = row0 + 8 * (r >> 2) + 4 * g + (r & 3) < N ? v[r] : 0.f;
    }
    if (diag) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool ok = __builtin_isfinite(v[r]);
        odd = odd || !ok;
        v[r] = ok ? v[r] : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i] = MFMA(v[r], w[r], acc[i]);
  }
  odd = __any(odd);
  if (odd) {
#pragma unroll
    for (int r = 0; r < 16; ++r) kept[(8 * (r >> 2) + 4 * g + (r & 3)) * 32 + c] = w[r];
  }
  return odd;
}
// the infinities and NaNs of a diagonal tile (row0 = its first row), for the columns that see them
template <int DH, class T, class Seen>
__device__ __forceinline__ void add_left_out(f32x16 (&acc)[DH / 32], const T *x, int64_t ld, int row0, int N, int dh, int c, int g, const float *kept, Seen seen) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // `kept` was written by this wave's other lanes
#pragma unroll 1
  for (int j = 0; j < 32 && row0 + j < N; ++j) {
    if (!seen(row0 + j)) continue;
    const float w = kept[j * 32 + c];
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int col = 32 * i + 8 * k + 4 * g;
        if (col >= dh) continue;
        const f32x4 v = get4(x + (int64_t)(row0 + j) * ld + col);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][4 * k + e] += __builtin_isfinite(v[e]) ? 0.f : v[e] * w;
      }
  }
}
template <int DH>
__device__ __forceinline__ void zero(f32x16 (&acc)[DH / 32]) {
#pragma unroll
  for (int i = 0; i < DH / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
}

// Sum of the NW waves' [dh][32] accumulators (each multiplied by its lane's `mul`) written as rows of `out` (stride ld) and, where it is
// given, unrounded to out32
template <int DH, int NW, class T>
__device__ __forceinline__ void merge(float *lds, const f32x16 (&acc)[DH / 32], float mul, T *out, float *out32, int64_t ld, int rows_left, int dh, int wave, int c, int g) {
  constexpr int LDR = DH + 4;
#pragma unroll
  for (int i = 0; i < DH / 32; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4 *>(lds + (wave * 32 + c) * LDR + 32 * i + 8 * j + 4 * g) =
          f32x4{acc[i][4 * j] * mul, acc[i][4 * j + 1] * mul, acc[i][4 * j + 2] * mul, acc[i][4 * j + 3] * mul};
  __syncthreads();
  constexpr int TPR = 2 * NW;  // threads per row
  const int row = threadIdx.x / TPR;
  if (row < rows_left)
    for (int k = threadIdx.x % TPR * 4; k < dh; k += 4 * TPR) {
      f32x4 v = *reinterpret_cast<const f32x4 *>(lds + row * LDR + k);
#pragma unroll
      for (int w = 1; w < NW; ++w) v += *reinterpret_cast<const f32x4 *>(lds + (w * 32 + row) * LDR + k);
      put4(out + row * ld + k, v);
      if (out32) put4(out32 + row * ld + k, v);
    }
  __syncthreads();
}

struct Item { int blk, b, h; };
// late query blocks (early key blocks) are the longest: they start first
__device__ __forceinline__ Item item_of(int N, int Hs, bool late_first) {
  const int nb = (N + 31) / 32, nbh = gridDim.x / nb, rank = (int)blockIdx.x / nbh, bh = (int)blockIdx.x % nbh;
  return {late_first ? nb - 1 - rank : rank, bh / Hs, bh % Hs};
}

template <int DH, int BF, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_fwd_kernel(const typename El<BF>::T *qkv, typename El<BF>::T *o, float *o32, float *lse, int N, int Hs, int dh, float scale, const int32_t *keep) {
  __shared__ __attribute__((aligned(16))) float lds[NW * 32 * (DH + 4)];
  __shared__ float ms[NW][32], ls[NW][32];
  const Item it = item_of(N, Hs, true);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int64_t HD = (int64_t)Hs * dh, ld = 3 * HD;
  const auto *qp = qkv + (int64_t)it.b * N * ld + (int64_t)it.h * dh, *kp = qp + HD, *vp = kp + HD;
  const int q0 = it.blk * 32, q = q0 + c;
  const float sc = scale * kLog2e;
  float *const kept = lds + wave * 32 * (DH + 4);  // the wave's part of the area that merge() uses afterwards
  bool left_out = false;
  const bool masked = keep && keep[it.h] < 0;  // masked head (Masked TwIST, Section 4.1): no key is visited, zeros are written
  f32x4 qf[DH / 8], kf[DH / 8];
  load_row<DH>(qf, qp + (int64_t)min(q, N - 1) * ld, dh, g);
  f32x16 acc[DH / 32];
  zero<DH>(acc);
  float m = -INFINITY, l = 0.f;
  for (int kt = wave; kt <= it.blk && !masked; kt += NW) {
    load_row<DH>(kf, kp + (int64_t)min(kt * 32 + c, N - 1) * ld, dh, g);
    f32x16 s = dot_tile<DH, kChains<BF>>(kf, qf);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (kt * 32 + 8 * (r >> 2) + 4 * g + (r & 3) > q) s[r] = -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), ref = mn == -INFINITY ? 0.f : mn;  // (all scores of the wave's tiles so far may be -inf: weights 0)
    const float alpha = fast_exp2((m - ref) * sc);
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = fast_exp2((s[r] - ref) * sc); sum += s[r]; }
    l = l * alpha + sum;
    m = mn;
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] *= alpha;
    left_out = add_tile<DH>(acc, vp, ld, kt * 32, N, dh, s, c, g, kt == it.blk, kept);
  }
  if (left_out) add_left_out<DH>(acc, vp, ld, q0, N, dh, c, g, kept, [&](int key) { return key <= q; });  // (a wave's last tile: no rescaling since)
  l += __shfl_xor(l, 32, 64);
  if (g == 0) { ms[wave][c] = m; ls[wave][c] = l; }
  __syncthreads();
  float mt = ms[0][c], lt = 0.f;
#pragma unroll
  for (int w = 1; w < NW; ++w) mt = fmaxf(mt, ms[w][c]);
#pragma unroll
  for (int w = 0; w < NW; ++w) lt += ls[w][c] * fast_exp2((ms[w][c] - mt) * sc);
  const float mul = masked ? 0.f : fast_exp2((m - mt) * sc) / lt;  // a wave without tiles has m = -inf: factor 0
  if (wave == 0 && g == 0 && q < N) lse[((int64_t)it.b * Hs + it.h) * N + q] = masked ? 0.f : fmaf(mt, scale, logf(lt));
  const int64_t at = ((int64_t)it.b * N + q0) * HD + (int64_t)it.h * dh;
  merge<DH, NW>(lds, acc, mul, o + at, o32 ? o32 + at : nullptr, HD, N - q0, dh, wave, c, g);
}

template <int DH, int BF, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_dq_kernel(const typename El<BF>::T *qkv, const typename El<BF>::T *dout, const float *o, const float *lse, float *delta,
                                                          typename El<BF>::T *dqkv, int N,
                                                          int Hs, int dh, float scale, const int32_t *keep) {
  __shared__ __attribute__((aligned(16))) float lds[NW * 32 * (DH + 4)];
  const Item it = item_of(N, Hs, true);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int64_t HD = (int64_t)Hs * dh, ld = 3 * HD;
  const auto *qp = qkv + (int64_t)it.b * N * ld + (int64_t)it.h * dh, *kp = qp + HD, *vp = kp + HD;
  const int q0 = it.blk * 32, q = q0 + c, qr = min(q, N - 1);
  float *const kept = lds + wave * 32 * (DH + 4);  // the wave's part of the area that merge() uses afterwards
  bool left_out = false;
  const int64_t row = ((int64_t)it.b * N + qr) * HD + (int64_t)it.h * dh, stat = ((int64_t)it.b * Hs + it.h) * N;
  const float L = lse[stat + qr];
  f32x4 qf[DH / 8], gf[DH / 8], kf[DH / 8];
  load_row<DH>(qf, qp + (int64_t)qr * ld, dh, g);
  load_row<DH>(gf, dout + row, dh, g);
  load_row<DH>(kf, o + row, dh, g);
  float dl = 0.f;
#pragma unroll
  for (int u = 0; u < DH / 8; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) dl += gf[u][e] * kf[u][e];
  dl += __shfl_xor(dl, 32, 64);
  if (wave == 0 && g == 0 && q < N) delta[stat + q] = dl;
  const bool masked = keep && keep[it.h] < 0;
  f32x16 acc[DH / 32];
  zero<DH>(acc);
  for (int kt = wave; kt <= it.blk && !masked; kt += NW) {
    const int64_t kr = min(kt * 32 + c, N - 1);
    load_row<DH>(kf, kp + kr * ld, dh, g);
    f32x16 s = dot_tile<DH, kChains<BF>>(kf, qf);
    load_row<DH>(kf, vp + kr * ld, dh, g);
    const f32x16 dp = dot_tile<DH, BF ? 1 : 2>(kf, gf);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float ds = fast_exp2(fmaf(s[r], scale, -L) * kLog2e) * (dp[r] - dl) * scale;
      s[r] = kt * 32 + 8 * (r >> 2) + 4 * g + (r & 3) > q ? 0.f : ds;
    }
    left_out = add_tile<DH>(acc, kp, ld, kt * 32, N, dh, s, c, g, kt == it.blk, kept);
  }
  if (left_out) add_left_out<DH>(acc, kp, ld, q0, N, dh, c, g, kept, [&](int key) { return key <= q; });
  merge<DH, NW>(lds, acc, 1.f, dqkv + ((int64_t)it.b * N + q0) * ld + (int64_t)it.h * dh, nullptr, ld, N - q0, dh, wave, c, g);
}

template <int DH, int BF, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_dkv_kernel(const typename El<BF>::T *qkv, const typename El<BF>::T *dout, const float *lse, const float *delta,
                                                           typename El<BF>::T *dqkv, int N, int Hs,
                                                           int dh, float scale, const int32_t *keep) {
  __shared__ __attribute__((aligned(16))) float lds[NW * 32 * (DH + 4)];
  // Eight waves have half the registers each: the key and value rows, the same for all, lie in LDS
  constexpr bool SHARED = NW == 8;
  constexpr int LDR = DH + 4;
  __shared__ __attribute__((aligned(16))) float rows[SHARED ? 2 * 32 * LDR : 4];
  __shared__ float kept[2][32 * 32];  // wave 0's, which has the diagonal tile
  const Item it = item_of(N, Hs, false);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int64_t HD = (int64_t)Hs * dh, ld = 3 * HD;
  const auto *qp = qkv + (int64_t)it.b * N * ld + (int64_t)it.h * dh, *kp = qp + HD, *vp = kp + HD;
  const auto *gp = dout + (int64_t)it.b * N * HD + (int64_t)it.h * dh;
  const int k0 = it.blk * 32, kv = k0 + c, kr = min(kv, N - 1);
  bool dv_left_out = false, dk_left_out = false;
  const float *lse_b = lse + ((int64_t)it.b * Hs + it.h) * N, *del_b = delta + ((int64_t)it.b * Hs + it.h) * N;
  const bool masked = keep && keep[it.h] < 0;
  f32x4 kf[DH / 8], vf[DH / 8], xf[DH / 8];
  const float *const ks = rows + c * LDR + 4 * g, *const vs = ks + 32 * LDR;
  if constexpr (SHARED) {
    if (wave < 2) {
      load_row<DH>(xf, (wave ? vp : kp) + (int64_t)kr * ld, dh, g);
#pragma unroll
      for (int u = 0; u < DH / 8; ++u) *reinterpret_cast<f32x4 *>(rows + (32 * wave + c) * LDR + 8 * u + 4 * g) = xf[u];
    }
    __syncthreads();
  } else {
    load_row<DH>(kf, kp + (int64_t)kr * ld, dh, g);
    load_row<DH>(vf, vp + (int64_t)kr * ld, dh, g);
  }
  f32x16 dk[DH / 32], dv[DH / 32];
  zero<DH>(dk);
  zero<DH>(dv);
  const int n_q = (N + 31) / 32;
  for (int qt = it.blk + wave; qt < n_q && !masked; qt += NW) {
    const int q0 = qt * 32;
    const int64_t qr = min(q0 + c, N - 1);
    load_row<DH>(xf, qp + qr * ld, dh, g);
    if constexpr (SHARED) asm volatile("" ::: "memory");  // (the rows in LDS are not to be kept in registers)
    f32x16 s;
    if constexpr (SHARED) s = dot_tile<DH, kChains<BF>>(xf, ks);
    else s = dot_tile<DH, kChains<BF>>(xf, kf);
    load_row<DH>(xf, gp + qr * HD, dh, g);
    f32x16 dp;
    if constexpr (SHARED) dp = dot_tile<DH, BF ? 1 : 2>(xf, vs);
    else dp = dot_tile<DH, BF ? 1 : 2>(xf, vf);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int q = q0 + 8 * (r >> 2) + 4 * g + (r & 3), qc = min(q, N - 1);
      const float p = fast_exp2(fmaf(s[r], scale, -lse_b[qc]) * kLog2e), ds = p * (dp[r] - del_b[qc]) * scale;
      const bool hidden = q < kv || q >= N;
      dp[r] = hidden ? 0.f : ds;
      s[r] = hidden ? 0.f : p;
    }
    dv_left_out = dv_left_out | add_tile<DH>(dv, gp, HD, q0, N, dh, s, c, g, qt == it.blk, kept[0]);
    dk_left_out = dk_left_out | add_tile<DH>(dk, qp, ld, q0, N, dh, dp, c, g, qt == it.blk, kept[1]);
  }
  auto seen = [&](int q) { return q >= kv; };
  if (dv_left_out) add_left_out<DH>(dv, gp, HD, k0, N, dh, c, g, kept[0], seen);
  if (dk_left_out) add_left_out<DH>(dk, qp, ld, k0, N, dh, c, g, kept[1], seen);
  auto *out = dqkv + ((int64_t)it.b * N + k0) * ld + HD + (int64_t)it.h * dh;
  merge<DH, NW>(lds, dk, 1.f, out, nullptr, ld, N - k0, dh, wave, c, g);
  merge<DH, NW>(lds, dv, 1.f, out + HD, nullptr, ld, N - k0, dh, wave, c, g);
}

bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// WG(DH, NW) for heads of up to DH columns and workgroups of NW waves
#define TW_F32_DH(dh, wide, WG)               \
  do {                                        \
    if ((dh) <= 32 && (wide)) WG(32, 8);      \
    else if ((dh) <= 32) WG(32, 4);           \
    else if ((dh) <= 64 && (wide)) WG(64, 8); \
    else if ((dh) <= 64) WG(64, 4);           \
    else WG(128, 4);                          \
  } while (0)

// Eight waves to a workgroup where there are few workgroups to a CU and more tiles of 32 in a sequence than four waves: the chain of a wave is half as
// long, and a second wave a SIMD works while the first waits for operands.  Forward / forward and backward, fp32, us, four waves and eight: 2 x 512
// tokens, 6 heads of 64 19.5 / 81.8 and 18.4 / 77.6; 1 x 2048, 6 of 64 (384 workgroups) 73 / 283 and 55 / 241; 1 x 4096, 4 of 32 (512) 86 / 346 and
// 63 / 275; 4 x 1024, 8 of 64 (1024) 69 / 332 and 72 / 312.  Of a short sequence's rows few see tiles for eight waves, and the others' wait in
// workgroups that share a CU: 160 tokens, 40 workgroups 11.9 / 48 and 11.8 / 43, 320 13 / 57 and 16 / 62, 480 14 / 71 and 19 / 73; 256 tokens, 192 12.6 / 50 and 13 / 50, 512
// 16 / 76 and 20 / 79; 288 tokens, 288 16.5 / 65 and 16 / 64, 504 20 / 90 and 22 / 89.  Heads of 128 do not fit the registers of a wave among eight.
static bool wide_of(int64_t workgroups, int N) { return N > 128 && workgroups <= (N <= 256 ? 256 : N <= 320 ? 384 : 512); }

bool twist_attention_f32_ok(const twist_ctx *ctx, const void *qkv, const void *o, const void *dout, const void *dqkv, int dh) {
  return !ctx->plain_only && dh % 4 == 0 && dh <= 128 && al16(qkv) && al16(o) && al16(dout) && al16(dqkv);
}

twist_status twist_attention_f32_fwd(twist_ctx *ctx, int bf16, const void *qkv, void *o, float *o32, float *lse, int B, int N, int Hs, int dh, const int32_t *keep) {
  const dim3 grid((unsigned)((int64_t)((N + 31) / 32) * B * Hs));
  const float scale = 1.0f / sqrtf((float)dh);
  const bool wide = wide_of(grid.x, N);
#define TW_FWD_BF(DH, NW) hipLaunchKernelGGL((attn_f32_fwd_kernel<DH, 1, NW>), grid, dim3(64 * NW), 0, ctx->stream, static_cast<const uint16_t *>(qkv), static_cast<uint16_t *>(o), o32, lse, N, Hs, dh, scale, keep)
#define TW_FWD(DH, NW) hipLaunchKernelGGL((attn_f32_fwd_kernel<DH, 0, NW>), grid, dim3(64 * NW), 0, ctx->stream, static_cast<const float *>(qkv), static_cast<float *>(o), nullptr, lse, N, Hs, dh, scale, keep)
  if (bf16) TW_F32_DH(dh, wide, TW_FWD_BF);
  else TW_F32_DH(dh, wide, TW_FWD);
#undef TW_FWD_BF
#undef TW_FWD
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

template <int BF>
static void launch_bwd(hipStream_t st, const void *qkv, const float *o, const void *dout, const float *lse, float *delta, void *dqkv, int B, int N, int Hs, int dh,
                       const int32_t *keep) {
  using T = typename El<BF>::T;
  const dim3 grid((unsigned)((int64_t)((N + 31) / 32) * B * Hs));
  const float scale = 1.0f / sqrtf((float)dh);
  const bool wide = wide_of(grid.x, N);
  const T *x = static_cast<const T *>(qkv), *gout = static_cast<const T *>(dout);
  T *dx = static_cast<T *>(dqkv);
#define TW_BWD(DH, NW)                                                                                                                                            \
  do {                                                                                                                                                               \
    hipLaunchKernelGGL((attn_f32_dq_kernel<DH, BF, NW>), grid, dim3(64 * NW), 0, st, x, gout, o, lse, delta, dx, N, Hs, dh, scale, keep);  \
    hipLaunchKernelGGL((attn_f32_dkv_kernel<DH, BF, NW>), grid, dim3(64 * NW), 0, st, x, gout, lse, delta, dx, N, Hs, dh, scale, keep);    \
  } while (0)
  TW_F32_DH(dh, wide, TW_BWD);
#undef TW_BWD
}

twist_status twist_attention_f32_bwd(twist_ctx *ctx, int bf16, const void *qkv, const float *o, const void *dout, const float *lse, float *delta, void *dqkv, int B, int N,
                                     int Hs, int dh, const int32_t *keep) {
  if (bf16) launch_bwd<1>(ctx->stream, qkv, o, dout, lse, delta, dqkv, B, N, Hs, dh, keep);
  else launch_bwd<0>(ctx->stream, qkv, o, dout, lse, delta, dqkv, B, N, Hs, dh, keep);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}
