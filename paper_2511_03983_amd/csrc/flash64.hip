// Causal attention of bf16 models on the matrix cores (v_mfma_f32_32x32x16_bf16) in workgroups of 64 queries or keys, forward and backward,
// d_head 32, 64 or 128.  TERMS = 3: probabilities and score gradients in fp32, any N.  TERMS = 1: rounded to bf16, as in flash.hip, for the forms of
// that file where 128-row workgroups are too few to fill the chip (few_rows in attention.hip).
//
// What bounded the former (flash_f32.hip: every product on the fp32 matrix instruction, at a sixteenth of the bf16 rate): the matrix
// pipes.  q, k, v and dO are bf16, so their products are exact in fp32 and S and dP belong on the bf16 instruction as they are.  A
// probability or a score gradient is fp32 and is fed to it as three bf16 terms of 8 bits each, whose sum is exactly the fp32 value
// (terms3); with a bf16 operand on the other side those products are exact as well, and only the order of sums differs from the fp32
// instruction.  Four bf16 products where there were two, at a sixteenth of the time each.
//
// Work is cut for few and short sequences, where the longest chain of dependent steps in a workgroup is what counts: a workgroup owns 64
// queries (forward, dQ) or 64 keys (dK / dV), and its four SIMDs are two groups of 32 of those times the two halves of every 64-row tile
// on the other side; the halves' results are added through LDS at the end, in fixed order.
//
// Layouts, swizzles and direct-to-LDS loads are those of flash.hip: S^T = K Q^T in the forward and dQ kernels (a lane owns a query), S = Q K^T
// in the dK / dV kernel (a lane owns a key), two 64-row tiles a stage.  The dK / dV kernel has a producer and a consumer wave per SIMD as there;
// P and dS are handed over in fp32 (TERMS = 3) and split by the consumer.
// Rows beyond N: as keys or queries of a tile they read as zeros (outside the buffer's range), in registers they are clamped to N - 1
// and their results not stored; a key beyond N comes after every query, a query beyond N gets probability zero.
// An infinity or a NaN reaches what depends on it and nothing else: hidden entries have weight zero, but zero times an infinity or a NaN is a
// NaN, so on diagonal tiles such values of the operand rows are left out of the products (clean), and where there was one, add_left_out
// adds what the columns do see of them.
//
// Measured (us, forward / forward and backward; before: the fp32 instruction):        error of the output in fp32, before in brackets
//   3 x 1000 tokens,  7 heads of 128     32 / 111   (128 / 563)                        1.55e-7 (1.87e-7)
//   2 x 500, 32 heads of 128             21 / 81    (104 / 461)                        1.36e-7 (1.66e-7)
//   2 x 3001, 16 heads of 128           168 / 712  (1203 / 5642)
//   8 x 1000, 3 heads of 64              22 / 76    (59 / 289)                         1.40e-7 (1.66e-7); scores of +-30 3.5e-7 (3.9e-7)
//   4 x 1024, 8 heads of 32              17 / 61    (41 / 174)
//   1 x 33, 4 heads of 64                11.5 / 19.5 (11.5 / 34)                       0.75e-7 (0.92e-7)
// 2 x 333, 3 heads of 64: 12 / 32.6 (17 / 71).  What bounds them now is the chain of steps in the longest workgroup.
#include <type_traits>

#include "flash_tile.h"

namespace {

constexpr uint32_t kOob = 0x80000000u;  // byte offset beyond every buffer (at most 2 GiB): loads return 0
#define WAIT_VM_LGKM0(vm) __builtin_amdgcn_s_waitcnt(0x0070 | ((vm) & 15) | ((vm) >> 4) << 14)  // vmcnt(vm < 64), lgkmcnt(0)

// v[r0 .. r0 + 7] as three vectors of bf16 that add up to it exactly: 8 bits of the mantissa each, cut off, not rounded (so that no value
// becomes infinite); an infinity is (infinity, 0, 0)
__device__ __forceinline__ void terms3(const f32x16 &v, int r0, bf16x8 (&t)[3]) {
  u32x4 w[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = v[r0 + 2 * e], b = v[r0 + 2 * e + 1];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
      w[k][e] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);  // the upper halves
      if (k == 2) break;
      a -= __uint_as_float(ua & 0xffff0000u);
      b -= __uint_as_float(ub & 0xffff0000u);
      if (k == 0) {
        a = a == a ? a : 0.f;
        b = b == b ? b : 0.f;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) t[k] = __builtin_bit_cast(bf16x8, w[k]);
}
// the weights v[r0 .. r0 + 7] as they are fed to the matrix instruction: exactly, in three terms, or rounded to bf16
template <int TERMS>
__device__ __forceinline__ void weights(const f32x16 &v, int r0, bf16x8 (&t)[TERMS]) {
  if constexpr (TERMS == 3) terms3(v, r0, t);
  else t[0] = pack8(v, r0);
}

// An operand fragment without its infinities and NaNs (`odd` becomes nonzero if there were any): exponents of all ones carry into the sign
__device__ __forceinline__ bf16x8 clean(bf16x8 f, uint32_t &odd) {
  u32x4 u = __builtin_bit_cast(u32x4, f);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t bad = ((u[e] & 0x7f807f80u) + 0x00800080u) & 0x80008000u;
    odd |= bad;
    u[e] &= ~(bad | (bad - (bad >> 15)));
  }
  return __builtin_bit_cast(bf16x8, u);
}
// acc[i][r] += weight(row) x[row][column 32 i + 8 (r / 4) + 4 g + r % 4] for the infinities and NaNs x among `rows` rows that seen(row)
template <int MT, class Seen, class Weight>
__device__ __forceinline__ void add_left_out(f32x16 (&acc)[MT], const uint16_t *x, int64_t ld, int rows, int g, Seen seen, Weight weight) {
#pragma unroll 1
  for (int j = 0; j < rows; ++j) {
    if (!seen(j)) continue;
    const float w = weight(j);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u32x2 u = *reinterpret_cast<const u32x2 *>(x + (int64_t)j * ld + 32 * i + 8 * k + 4 * g);
        const float v[4] = {__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][4 * k + e] += __builtin_isfinite(v[e]) ? 0.f : v[e] * w;
        __builtin_amdgcn_sched_barrier(0);  // (a rare path: few registers rather than loads in flight)
      }
  }
}

// one row's fragments for the contraction along d_head
template <int KS>
__device__ __forceinline__ void load_row(bf16x8 (&f)[KS], const uint16_t *row, int g) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) f[ks] = *reinterpret_cast<const bf16x8 *>(row + ks * 16 + g * 8);
}
template <int MT>
__device__ __forceinline__ void zero(f32x16 (&acc)[MT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
}
// accumulators (lane: column c; registers: head-dim rows) to and from rows of DH + 4 floats
template <int MT>
__device__ __forceinline__ void put_rows(float *row, const f32x16 (&acc)[MT], int g) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<f32x4 *>(row + 32 * i + 8 * k + 4 * g) = f32x4{acc[i][4 * k], acc[i][4 * k + 1], acc[i][4 * k + 2], acc[i][4 * k + 3]};
}
template <int MT>
__device__ __forceinline__ void add_rows(f32x16 (&acc)[MT], const float *row, int g) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(row + 32 * i + 8 * k + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][4 * k + e] += v[e];
    }
}
template <int MT>
__device__ __forceinline__ void store_rows(uint16_t *out, float *out32, const f32x16 (&acc)[MT], int g) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int col = 32 * i + 8 * k + 4 * g;
      *reinterpret_cast<u32x2 *>(out + col) = u32x2{pack2(acc[i][4 * k], acc[i][4 * k + 1]), pack2(acc[i][4 * k + 2], acc[i][4 * k + 3])};
      if (out32) *reinterpret_cast<f32x4 *>(out32 + col) = f32x4{acc[i][4 * k], acc[i][4 * k + 1], acc[i][4 * k + 2], acc[i][4 * k + 3]};
    }
}

// the wave's 32 x 32 weights kept for add_left_out: register r of lane (g, c) is row 8 (r / 4) + 4 g + r % 4, column c
__device__ __forceinline__ void keep_weights(float *kept, const f32x16 &w, int c, int g) {
#pragma unroll
  for (int r = 0; r < 16; ++r) kept[(8 * (r >> 2) + 4 * g + (r & 3)) * 32 + c] = w[r];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // read by the wave's other lanes
}

// Late query blocks (early key blocks) are the longest.  Up to two workgroups a CU they are all resident and the two that share a CU should
// add up to the same (snake order); beyond that the longest start first.
__device__ __forceinline__ int rank_of(int b, int nwg) { return nwg <= 512 ? snake_rank(b, nwg) : b; }

template <int DH, int TERMS, int NST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attn64_fwd_kernel(const uint16_t *qkv, uint16_t *o, float *o32, float *lse, int N, int Hs,
                                                                                               float scale, const int32_t *keep) {
  using G = Geo<DH>;
  constexpr int KS = G::KS, MT = G::MT, TILE_B = G::TILE_B, STAGE_B = G::STAGE_B, RB = G::RB, LDR = DH + 4;
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE_B];
  static_assert(2 * 32 * LDR * 4 + 1024 <= NST * STAGE_B, "the halves are merged in the stages");
  const int nqb = (N + 63) / 64, nbh = gridDim.x / nqb;
  const int rank = rank_of(blockIdx.x, gridDim.x);
  const int qb = nqb - 1 - rank / nbh, bh = rank % nbh, b = bh / Hs, h = bh % Hs;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int qg = wave & 1, kg = wave >> 1;  // which 32 queries, which half of a key tile
  const int64_t HD = (int64_t)Hs * DH, ld = 3 * HD;
  const uint16_t *batch = qkv + (int64_t)b * N * ld, *qp = batch + (int64_t)h * DH, *vp = qp + 2 * HD;
  const int q0 = qb * 64 + 32 * qg, q = q0 + c;
  const float sc = scale * kLog2e;
  const desc_t rs = make_desc(batch, (uint32_t)(N * ld * 2));
  const uint32_t tstep = (uint32_t)(64 * ld * 2);
  TileLoader<DH> lk, lv;
  lk.init(ld, (uint32_t)((HD + h * DH) * 2), wave, lane);
  lv.init(ld, (uint32_t)((2 * HD + h * DH) * 2), wave, lane);
  ReadOffsets<DH> ro;
  ro.init(lane);
  const bool masked = keep && keep[h] < 0;  // masked head (Masked TwIST, Section 4.1): no key is visited, zeros are written
  const int n_tiles = masked ? 0 : qb + 1;
  auto issue = [&](int kt) {  // (beyond the last tile nothing is fetched, zeros are filled in)
    char *st = smem + kt % NST * STAGE_B;
    const uint32_t o = kt < n_tiles ? (uint32_t)kt * tstep : kOob;
    lk.issue(rs, st, o, wave);
    lv.issue(rs, st + TILE_B, o, wave);
  };
#pragma unroll
  for (int kt = 0; kt < NST - 1; ++kt) issue(kt);

  bf16x8 qf[KS];
  load_row<KS>(qf, qp + (int64_t)min(q, N - 1) * ld, g);
  f32x16 acc[MT];
  zero<MT>(acc);
  float m = -INFINITY, l = 0.f;  // of this wave's keys; m in units of unscaled scores
  // the wave's 32 keys from k0 on, at Kt and Vt
  auto body = [&](const char *Kt, const char *Vt, int k0, auto diag_c) {
    constexpr bool DIAG = decltype(diag_c)::value;
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = MFMA(frag(Kt, ro.fo[ks]), qf[ks], s);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (DIAG && k0 + 8 * (r >> 2) + 4 * g + (r & 3) > q) s[r] = -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // the reference is the largest score so far (one that lags behind would do for the range, but rounds the exponents of the largest
    // weights: error of the output 1.9e-7 instead of 1.55e-7, for 4 % of the time)
    const float mn = fmaxf(m, mx), ref = mn == -INFINITY ? 0.f : mn;  // (all scores so far may be -inf: weights 0)
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = fast_exp2((s[r] - ref) * sc);
      if (TERMS == 1 && r % 2) {  // the sum is that of the rounded weights, so that the output is an exact convex combination of the value rows
        const uint32_t u = pack2(s[r - 1], s[r]);
        sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u), __builtin_bit_cast(bf16x2, 0x3f803f80u), sum, false);
      }
      if (TERMS == 3) sum += s[r];
    }
    if (__any(mn > m)) {
      const float alpha = mn > m ? fast_exp2((m - ref) * sc) : 1.f;
      l *= alpha;
      m = mn;
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] *= alpha;
    }
    l += sum;
    uint32_t odd = 0u;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bf16x8 p[TERMS];
      weights<TERMS>(s, 8 * t, p);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        bf16x8 v = frag_tr(Vt + 16 * t * RB, ro.ta[i], ro.tb[i]);
        if (DIAG) v = clean(v, odd);
#pragma unroll
        for (int k = TERMS - 1; k >= 0; --k) acc[i] = MFMA(v, p[k], acc[i]);
      }
    }
    if (DIAG && __any(odd != 0u)) {
      const int after = (k0 >> 6) + 1 + wave * 4096 / STAGE_B;  // (the stages behind the last tile's are free)
      float *kept = reinterpret_cast<float *>(smem + after % NST * STAGE_B + wave * 4096 % STAGE_B);
      keep_weights(kept, s, c, g);
      add_left_out<MT>(acc, vp + (int64_t)k0 * ld, ld, min(32, N - k0), g, [&](int j) { return k0 + j <= q; }, [&](int j) { return kept[j * 32 + c]; });
    }
  };
  int kt = 0;
  for (; kt + 1 < n_tiles; ++kt) {
    WAIT_VM_LGKM0((NST - 2) * 2 * TileLoader<DH>::NP);  // this wave's pieces of tile kt have landed, its reads of the tile before have returned
    __builtin_amdgcn_s_barrier();                       // everybody's: tile kt can be read, the stage of the one before be overwritten
    issue(kt + NST - 1);
    const char *Kt = smem + kt % NST * STAGE_B + kg * 32 * RB;
    body(Kt, Kt + TILE_B, kt * 64 + 32 * kg, std::false_type());
  }
  WAIT_VM_LGKM0(0);
  __builtin_amdgcn_s_barrier();
  if (n_tiles && kg <= qg) {  // the last tile: keys 32 .. 63 of it are in the future of queries 0 .. 31
    const char *Kt = smem + kt % NST * STAGE_B + kg * 32 * RB;
    body(Kt, Kt + TILE_B, kt * 64 + 32 * kg, std::true_type());
  }
  DL_WAIT_LGKM0;
  __builtin_amdgcn_s_barrier();  // the stages are free
  l += __shfl_xor(l, 32, 64);
  float *ms = reinterpret_cast<float *>(smem + NST * STAGE_B - 1024), *ls = ms + 128;
  if (g == 0) { ms[wave * 32 + c] = m; ls[wave * 32 + c] = l; }
  __syncthreads();
  const float mo = ms[(wave ^ 2) * 32 + c], lo = ls[(wave ^ 2) * 32 + c];
  const float mt = fmaxf(m, mo), ref = mt == -INFINITY ? 0.f : mt, mine = fast_exp2((m - ref) * sc);
  const float lt = kg ? lo * fast_exp2((mo - ref) * sc) + l * mine : l * mine + lo * fast_exp2((mo - ref) * sc);
  const float mul = masked ? 0.f : mine / lt;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] *= mul;
  float *row = reinterpret_cast<float *>(smem) + (qg * 32 + c) * LDR;
  if (kg) put_rows<MT>(row, acc, g);
  __syncthreads();
  if (kg || q >= N) return;
  add_rows<MT>(acc, row, g);
  const int64_t at = ((int64_t)b * N + q) * HD + (int64_t)h * DH;
  store_rows<MT>(o + at, o32 ? o32 + at : nullptr, acc, g);
  if (g == 0) lse[((int64_t)b * Hs + h) * N + q] = masked ? 0.f : fmaf(mt, scale, logf(lt));
}

// delta_q = dO_q . O_q from the unrounded forward output, dS^T = p (dp - delta) scale, dQ^T[dh][q] += K^T[dh][kv] dS^T[kv][q]
template <int DH, int TERMS, int NST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attn64_dq_kernel(const uint16_t *qkv, const uint16_t *dout, const float *o32, const float *lse, float *delta,
                                                                                              uint16_t *dqkv, int N, int Hs, float scale, const float *rope, const int32_t *keep) {
  using G = Geo<DH>;
  constexpr int KS = G::KS, MT = G::MT, TILE_B = G::TILE_B, STAGE_B = G::STAGE_B, RB = G::RB, LDR = DH + 4;
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE_B];
  static_assert(2 * 32 * LDR * 4 + 1024 <= NST * STAGE_B, "the halves are merged in the stages");
  const int nqb = (N + 63) / 64, nbh = gridDim.x / nqb;
  const int rank = rank_of(blockIdx.x, gridDim.x);
  const int qb = nqb - 1 - rank / nbh, bh = rank % nbh, b = bh / Hs, h = bh % Hs;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int qg = wave & 1, kg = wave >> 1;
  const int64_t HD = (int64_t)Hs * DH, ld = 3 * HD;
  const uint16_t *batch = qkv + (int64_t)b * N * ld, *qp = batch + (int64_t)h * DH, *kp = qp + HD;
  const int q0 = qb * 64 + 32 * qg, q = q0 + c, qr = min(q, N - 1);
  const desc_t rs = make_desc(batch, (uint32_t)(N * ld * 2));
  const uint32_t tstep = (uint32_t)(64 * ld * 2);
  TileLoader<DH> lk, lv;
  lk.init(ld, (uint32_t)((HD + h * DH) * 2), wave, lane);
  lv.init(ld, (uint32_t)((2 * HD + h * DH) * 2), wave, lane);
  ReadOffsets<DH> ro;
  ro.init(lane);
  const bool masked = keep && keep[h] < 0;  // masked head: the gradient is zero, nothing is loaded
  const int n_tiles = masked ? 0 : qb + 1;
  auto issue = [&](int kt) {  // (beyond the last tile nothing is fetched, zeros are filled in)
    char *st = smem + kt % NST * STAGE_B;
    const uint32_t o = kt < n_tiles ? (uint32_t)kt * tstep : kOob;
    lk.issue(rs, st, o, wave);
    lv.issue(rs, st + TILE_B, o, wave);
  };
#pragma unroll
  for (int kt = 0; kt < NST - 1; ++kt) issue(kt);

  const int64_t at = ((int64_t)b * N + qr) * HD + (int64_t)h * DH, stat = ((int64_t)b * Hs + h) * N + qr;
  const float L = lse[stat];
  bf16x8 qf[KS], gf[KS];
  load_row<KS>(qf, qp + (int64_t)qr * ld, g);
  load_row<KS>(gf, dout + at, g);
  float dl = 0.f;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int k = ks * 16 + g * 8;
    const f32x4 oa = *reinterpret_cast<const f32x4 *>(o32 + at + k), ob = *reinterpret_cast<const f32x4 *>(o32 + at + k + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) dl += (float)gf[ks][e] * oa[e] + (float)gf[ks][e + 4] * ob[e];
  }
  dl += __shfl_xor(dl, 32, 64);
  if (kg == 0 && g == 0 && q < N) delta[stat] = dl;
  f32x16 acc[MT];
  zero<MT>(acc);
  auto body = [&](const char *Kt, const char *Vt, int k0, auto diag_c) {
    constexpr bool DIAG = decltype(diag_c)::value;
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      s = MFMA(frag(Kt, ro.fo[ks]), qf[ks], s);
      dp = MFMA(frag(Vt, ro.fo[ks]), gf[ks], dp);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float ds = fast_exp2(fmaf(s[r], scale, -L) * kLog2e) * (dp[r] - dl) * scale;
      s[r] = DIAG && k0 + 8 * (r >> 2) + 4 * g + (r & 3) > q ? 0.f : ds;
    }
    uint32_t odd = 0u;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bf16x8 d[TERMS];
      weights<TERMS>(s, 8 * t, d);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        bf16x8 k = frag_tr(Kt + 16 * t * RB, ro.ta[i], ro.tb[i]);
        if (DIAG) k = clean(k, odd);
#pragma unroll
        for (int e = TERMS - 1; e >= 0; --e) acc[i] = MFMA(k, d[e], acc[i]);
      }
    }
    if (DIAG && __any(odd != 0u)) {
      const int after = (k0 >> 6) + 1 + wave * 4096 / STAGE_B;  // (the stages behind the last tile's are free)
      float *kept = reinterpret_cast<float *>(smem + after % NST * STAGE_B + wave * 4096 % STAGE_B);
      keep_weights(kept, s, c, g);
      add_left_out<MT>(acc, kp + (int64_t)k0 * ld, ld, min(32, N - k0), g, [&](int j) { return k0 + j <= q; }, [&](int j) { return kept[j * 32 + c]; });
    }
  };
  int kt = 0;
  for (; kt + 1 < n_tiles; ++kt) {
    WAIT_VM_LGKM0((NST - 2) * 2 * TileLoader<DH>::NP);  // this wave's pieces of tile kt have landed, its reads of the tile before have returned
    __builtin_amdgcn_s_barrier();                       // everybody's: tile kt can be read, the stage of the one before be overwritten
    issue(kt + NST - 1);
    const char *Kt = smem + kt % NST * STAGE_B + kg * 32 * RB;
    body(Kt, Kt + TILE_B, kt * 64 + 32 * kg, std::false_type());
  }
  WAIT_VM_LGKM0(0);
  __builtin_amdgcn_s_barrier();
  if (n_tiles && kg <= qg) {  // the last tile: keys 32 .. 63 of it are in the future of queries 0 .. 31
    const char *Kt = smem + kt % NST * STAGE_B + kg * 32 * RB;
    body(Kt, Kt + TILE_B, kt * 64 + 32 * kg, std::true_type());
  }
  DL_WAIT_LGKM0;
  __builtin_amdgcn_s_barrier();
  float *row = reinterpret_cast<float *>(smem) + (qg * 32 + c) * LDR;
  if (kg) put_rows<MT>(row, acc, g);
  __syncthreads();
  if (kg || q >= N) return;
  add_rows<MT>(acc, row, g);
  if (DH >= 64 && rope) rope_grad<DH>(acc, rope, q, g);
  store_rows<MT>(dqkv + ((int64_t)b * N + q) * ld + (int64_t)h * DH, nullptr, acc, g);
}

// dV^T[dh][kv] += dO^T[dh][q] P[q][kv], dK^T[dh][kv] += Q^T[dh][q] dS[q][kv].  Wave w (producer) and w + 4 (consumer) share SIMD w: 32 keys
// (w & 1) and 32 queries (w >> 1) of every 64-query tile.  Three stages (the tile being loaded, the producer's, the consumer's, which is one
// behind), two hand-over areas; all of the CU's 160 KB at d_head 128, so the log-sum-exps and deltas travel in registers, a tile ahead.
template <int DH, int TERMS, int NST>
__global__ __launch_bounds__(512) void attn64_dkv_kernel(const uint16_t *qkv, const uint16_t *dout, const float *lse, const float *delta, uint16_t *dqkv, int N, int Hs,
                                                         float scale, const float *rope, const int32_t *keep) {
  using G = Geo<DH>;
  constexpr int KS = G::KS, MT = G::MT, TILE_B = G::TILE_B, STAGE_B = G::STAGE_B, RB = G::RB, LDR = DH + 4;
  constexpr int XCH = NST * STAGE_B;           // [2 tiles][4 SIMDs][P, dS][4 register quads, or 2 octets in bf16][64 lanes] x 16 bytes
  constexpr int XB = TERMS == 3 ? 8192 : 4096;
  constexpr bool LDS_STATS = NST > 3;          // the log-sum-exps and deltas of a tile, 512 bytes a stage
  constexpr int STATS = XCH + 2 * 4 * XB;
  __shared__ __attribute__((aligned(1024))) char smem[STATS + (LDS_STATS ? NST * 512 : 0)];
  static_assert(4 * 32 * LDR * 4 <= XCH + 2 * 4 * XB, "the halves are merged in the stages");
  const int nkb = (N + 63) / 64, nbh = gridDim.x / nkb;
  const int kb = (int)blockIdx.x / nbh, bh = (int)blockIdx.x % nbh, b = bh / Hs, h = bh % Hs;  // early key blocks are the longest: they start first
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
  const int simd = wave & 3, kg = simd & 1, qg = simd >> 1;
  const bool producer = wave < 4;
  const int64_t HD = (int64_t)Hs * DH, ld = 3 * HD;
  const uint16_t *batch = qkv + (int64_t)b * N * ld, *qp = batch + (int64_t)h * DH;
  const uint16_t *gbatch = dout + (int64_t)b * N * HD, *gp = gbatch + (int64_t)h * DH;
  const float *lse_b = lse + ((int64_t)b * Hs + h) * N, *del_b = delta + ((int64_t)b * Hs + h) * N;
  const desc_t rq = make_desc(batch, (uint32_t)(N * ld * 2)), rg = make_desc(gbatch, (uint32_t)(N * HD * 2));
  const uint32_t qstep = (uint32_t)(64 * ld * 2), gstep = (uint32_t)(64 * HD * 2);
  TileLoader<DH> lt;  // the producers bring in the query tiles, the consumers the dO tiles
  if (producer) lt.init(ld, (uint32_t)(h * DH * 2), simd, lane);
  else lt.init(HD, (uint32_t)(h * DH * 2), simd, lane);
  ReadOffsets<DH> ro;
  ro.init(lane);
  const bool masked = keep && keep[h] < 0;  // masked head: the gradients are zero, nothing is loaded
  const int k0 = kb * 64 + 32 * kg, kv = k0 + c, kr = min(kv, N - 1);
  const int n_ph = masked ? 0 : nkb - kb;   // query tiles at or below the diagonal
  const desc_t rst = make_desc(producer ? lse_b : del_b, (uint32_t)(N * 4));
  auto issue = [&](int ph) {  // (beyond the last tile nothing is fetched, zeros are filled in)
    char *st = smem + ph % NST * STAGE_B;
    const bool in = ph < n_ph;
    if (producer) lt.issue(rq, st, in ? (uint32_t)(kb + ph) * qstep : kOob, simd);
    else lt.issue(rg, st + TILE_B, in ? (uint32_t)(kb + ph) * gstep : kOob, simd);
    if (LDS_STATS && simd == 0) dma<4>(rst, smem + STATS + ph % NST * 512 + (producer ? 0 : 256), in ? (uint32_t)((kb + ph) * 256 + lane * 4) : kOob);
  };
  // all but the loads of the newest PF - 1 tiles have landed; LDS reads have returned, writes are done
  constexpr int PF = NST - 2, NP = TileLoader<DH>::NP;
  auto wait = [&] {
    if (LDS_STATS && simd == 0) WAIT_VM_LGKM0((PF - 1) * (NP + 1));
    else WAIT_VM_LGKM0((PF - 1) * NP);
  };
  // tile 0 is on the diagonal: there SIMD (kg 1, qg 0) has nothing, (0, 1) everything, the others a triangle
  const bool idle = kg > qg;
#pragma unroll
  for (int ph = 0; ph < PF; ++ph) issue(ph);
  if (producer) {
    bf16x8 kf[KS], vf[KS];
    load_row<KS>(kf, qp + HD + (int64_t)kr * ld, g);
    load_row<KS>(vf, qp + 2 * HD + (int64_t)kr * ld, g);
    // log-sum-exp and delta of the lane's 16 query rows, a tile ahead
    f32x4 L[4], D[4], Ln[4], Dn[4];
    auto stats = [&](int ph) {
      const int q0 = (kb + ph) * 64 + 32 * qg;
      typedef f32x4 __attribute__((aligned(4))) f32x4u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int q = q0 + 8 * k + 4 * g;
        if (q0 + 32 <= N) {
          Ln[k] = *reinterpret_cast<const f32x4u *>(lse_b + q);
          Dn[k] = *reinterpret_cast<const f32x4u *>(del_b + q);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) { Ln[k][e] = lse_b[min(q + e, N - 1)]; Dn[k][e] = del_b[min(q + e, N - 1)]; }
        }
      }
    };
    if (!LDS_STATS && n_ph) stats(0);
    DL_WAIT_VM0;  // the first tiles, and the key / value fragments
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));  // (used here: the compiler may not sink the loads, and its waits for them, into the loop)
    __builtin_amdgcn_s_barrier();
    for (int ph = 0; ph <= n_ph; ++ph) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (LDS_STATS) {
          const char *st = smem + STATS + ph % NST * 512 + (32 * qg + 8 * k + 4 * g) * 4;
          L[k] = *reinterpret_cast<const f32x4 *>(st);
          D[k] = *reinterpret_cast<const f32x4 *>(st + 256);
        } else {
          L[k] = Ln[k];
          D[k] = Dn[k];
        }
      }
      if (!LDS_STATS && ph + 1 < n_ph) stats(ph + 1);
      issue(ph + PF);
      if (ph < n_ph && !(idle && ph == 0)) {
        const char *Qt = smem + ph % NST * STAGE_B + qg * 32 * RB, *Gt = Qt + TILE_B;
        f32x16 s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          s = MFMA(frag(Qt, ro.fo[ks]), kf[ks], s);
          dp = MFMA(frag(Gt, ro.fo[ks]), vf[ks], dp);
        }
        const int q0 = (kb + ph) * 64 + 32 * qg;
        const bool edge = q0 == k0 || q0 + 32 > N;  // some query precedes a key, or is beyond the sequence
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int q = q0 + 8 * (r >> 2) + 4 * g + (r & 3);
          const bool hidden = edge && (q < kv || q >= N);
          const float p = fast_exp2(fmaf(s[r], scale, -L[r >> 2][r & 3]) * kLog2e), ds = p * (dp[r] - D[r >> 2][r & 3]) * scale;
          dp[r] = hidden ? 0.f : ds;
          s[r] = hidden ? 0.f : p;
        }
        char *X = smem + XCH + ((ph & 1) * 4 + simd) * XB + 16 * lane;
        if (TERMS == 3) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            *reinterpret_cast<f32x4 *>(X + 1024 * k) = f32x4{s[4 * k], s[4 * k + 1], s[4 * k + 2], s[4 * k + 3]};
            *reinterpret_cast<f32x4 *>(X + 4096 + 1024 * k) = f32x4{dp[4 * k], dp[4 * k + 1], dp[4 * k + 2], dp[4 * k + 3]};
          }
        } else {
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            *reinterpret_cast<bf16x8 *>(X + 1024 * k) = pack8(s, 8 * k);
            *reinterpret_cast<bf16x8 *>(X + 2048 + 1024 * k) = pack8(dp, 8 * k);
          }
        }
      }
      wait();  // this wave's pieces of the next tile have landed, the hand-over is written
      __builtin_amdgcn_s_barrier();
    }
    DL_WAIT_VM0;
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_s_barrier();  // (the consumers' exchange below)
  } else {
    f32x16 dk[MT], dv[MT];
    zero<MT>(dk);
    zero<MT>(dv);
    DL_WAIT_VM0;
    __builtin_amdgcn_s_barrier();
    auto body = [&](int pp, auto diag_c) {
      constexpr bool DIAG = decltype(diag_c)::value;
      const char *Qt = smem + pp % NST * STAGE_B + qg * 32 * RB, *Gt = Qt + TILE_B;
      const char *X = smem + XCH + ((pp & 1) * 4 + simd) * XB;
      uint32_t odd_v = 0u, odd_k = 0u;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        bf16x8 pt[TERMS], dt[TERMS];
        if constexpr (TERMS == 3) {
          f32x16 w;  // P, dS of the lane's 8 rows of this half
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(X + (k >> 1) * 4096 + (2 * t + (k & 1)) * 1024 + 16 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[4 * k + e] = x[e];
          }
          terms3(w, 0, pt);
          terms3(w, 8, dt);
        } else {
          pt[0] = *reinterpret_cast<const bf16x8 *>(X + t * 1024 + 16 * lane);
          dt[0] = *reinterpret_cast<const bf16x8 *>(X + 2048 + t * 1024 + 16 * lane);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          bf16x8 x = frag_tr(Gt + 16 * t * RB, ro.ta[i], ro.tb[i]), y = frag_tr(Qt + 16 * t * RB, ro.ta[i], ro.tb[i]);
          if (DIAG) {
            x = clean(x, odd_v);
            y = clean(y, odd_k);
          }
#pragma unroll
          for (int k = TERMS - 1; k >= 0; --k) {
            dv[i] = MFMA(x, pt[k], dv[i]);
            dk[i] = MFMA(y, dt[k], dk[i]);
          }
        }
      }
      if (DIAG) {
        const int q0 = (kb + pp) * 64 + 32 * qg, rows = min(32, N - q0);
        auto seen = [&](int j) { return q0 + j >= kv; };
        auto at = [&](int part, int j) {  // P or dS of row j, register 4 (j / 8) + j % 4 of half j / 4 % 2, and the lane's column
          const int r = 4 * (j >> 3) + (j & 3), l = ((j >> 2) & 1) * 32 + c;
          if (TERMS == 3) return *reinterpret_cast<const float *>(X + part * 4096 + (r >> 2) * 1024 + 16 * l + 4 * (r & 3));
          return __uint_as_float((uint32_t)*reinterpret_cast<const uint16_t *>(X + part * 2048 + (r >> 3) * 1024 + 16 * l + 2 * (r & 7)) << 16);
        };
        if (__any(odd_v != 0u)) add_left_out<MT>(dv, gp + (int64_t)q0 * HD, HD, rows, g, seen, [&](int j) { return at(0, j); });
        if (__any(odd_k != 0u)) add_left_out<MT>(dk, qp + (int64_t)q0 * ld, ld, rows, g, seen, [&](int j) { return at(1, j); });
      }
    };
    auto phase = [&](int ph, auto work) {
      issue(ph + PF);
      work();
      wait();  // ... and every LDS read of the tile has returned before the stage and the hand-over area are released
      __builtin_amdgcn_s_barrier();
    };
    phase(0, [] {});
    if (n_ph) phase(1, [&] { if (!idle) body(0, std::true_type()); });
    for (int ph = 2; ph <= n_ph; ++ph) phase(ph, [&] { body(ph - 1, std::false_type()); });
    DL_WAIT_VM0;                   // the zero fills beyond the last tile
    __builtin_amdgcn_s_barrier();  // everybody's
    // the two query halves are added: the consumers of the first finish dK, those of the second dV
    float *rows = reinterpret_cast<float *>(smem) + (kg * 32 + c) * LDR;  // dV of the first half; 64 rows further: dK of the second
    if (qg == 0) put_rows<MT>(rows, dv, g);
    else put_rows<MT>(rows + 64 * LDR, dk, g);
    DL_WAIT_LGKM0;
    __builtin_amdgcn_s_barrier();
    if (kv >= N) return;
    uint16_t *out = dqkv + ((int64_t)b * N + kv) * ld + HD + (int64_t)h * DH;
    if (qg == 0) {
      add_rows<MT>(dk, rows + 64 * LDR, g);
      if (DH >= 64 && rope) rope_grad<DH>(dk, rope, kv, g);
      store_rows<MT>(out, nullptr, dk, g);
    } else {
      add_rows<MT>(dv, rows, g);
      store_rows<MT>(out + HD, nullptr, dv, g);
    }
  }
}

bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// runs `expr` with DH standing for the head width, TERMS for the terms of a weight, NSQ and NSK for the stages of the forward and dQ kernels
// and of the dK / dV kernel.  64- and 32-wide heads: a few more stages than two and three are free and save the backward kernels up to 14 %
// (1 x 2048 tokens, 8 heads of 64: 66.8 -> 57.7 us); 128-wide ones: four stages leave one forward or dQ workgroup on a CU
// (1 x 4096, 4 heads: 74 -> 91 us).
#define TW_DH64(dh, rounded, expr)                                                                       \
  do {                                                                                                   \
    if ((dh) == 32) { constexpr int DH = 32, TERMS = 3, NSQ = 4, NSK = 5; expr; }                        \
    else if ((dh) == 64 && !(rounded)) { constexpr int DH = 64, TERMS = 3, NSQ = 4, NSK = 5; expr; }     \
    else if ((dh) == 64) { constexpr int DH = 64, TERMS = 1, NSQ = 4, NSK = 5; expr; }                   \
    else if (!(rounded)) { constexpr int DH = 128, TERMS = 3, NSQ = 2, NSK = 3; expr; }                  \
    else { constexpr int DH = 128, TERMS = 1, NSQ = 2, NSK = 3; expr; }                                  \
  } while (0)

// Everything in bf16 with these head widths that flash.hip does not take; faster than flash_f32.hip at every size tried (figures above).
// A batch element has to lie in one 32-bit buffer range.
bool twist_attention_64_ok(const twist_ctx *ctx, const void *qkv, const void *o, const void *o32, const void *dout, const void *dqkv, int N, int Hs, int dh) {
  return !ctx->plain_only && (dh == 32 || dh == 64 || dh == 128) && (int64_t)N * 3 * Hs * dh * 2 < (1ll << 31) && al16(qkv) && al16(o) && al16(o32) && al16(dout) && al16(dqkv);
}

twist_status twist_attention_64_fwd(twist_ctx *ctx, const void *qkv, void *o, float *o32, float *lse, int B, int N, int Hs, int dh, const int32_t *keep, bool rounded) {
  const dim3 grid((unsigned)((int64_t)((N + 63) / 64) * B * Hs)), block(256);
  TW_DH64(dh, rounded, hipLaunchKernelGGL((attn64_fwd_kernel<DH, TERMS, NSQ>), grid, block, 0, ctx->stream, static_cast<const uint16_t *>(qkv), static_cast<uint16_t *>(o), o32, lse, N, Hs,
                                 1.0f / sqrtf((float)dh), keep));
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_attention_64_bwd(twist_ctx *ctx, const void *qkv, const float *o32, const void *dout, const float *lse, float *delta, void *dqkv, int B, int N, int Hs, int dh,
                                    const float *rope_tab, const int32_t *keep, bool rounded, bool *rope_done) {
  const dim3 grid((unsigned)((int64_t)((N + 63) / 64) * B * Hs));
  const float scale = 1.0f / sqrtf((float)dh);
  const uint16_t *x = static_cast<const uint16_t *>(qkv), *gout = static_cast<const uint16_t *>(dout);
  uint16_t *dx = static_cast<uint16_t *>(dqkv);
  const float *rt = rope_tab && al16(rope_tab) && dh >= 64 ? rope_tab : nullptr;
  TW_DH64(dh, rounded, hipLaunchKernelGGL((attn64_dq_kernel<DH, TERMS, NSQ>), grid, dim3(256), 0, ctx->stream, x, gout, o32, lse, delta, dx, N, Hs, scale, rt, keep);
          hipLaunchKernelGGL((attn64_dkv_kernel<DH, TERMS, NSK>), grid, dim3(512), 0, ctx->stream, x, gout, lse, delta, dx, N, Hs, scale, rt, keep));
  TW_HIP(ctx, hipGetLastError());
  *rope_done = rt != nullptr;
  return TWIST_OK;
}
