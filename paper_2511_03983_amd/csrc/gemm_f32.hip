// Dense projections of fp32 models on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: exact fp32 products, fp32
// accumulation, the same precision as the vector units at the matrix pipes' issue rate).
//
// Workgroup tile BM x BN, four waves, the contraction walked in slices of BK that are double-buffered in LDS (the next slice's
// global loads are in flight while the current one is multiplied, one barrier per slice).  The waves divide the tile (WK = 1), or
// the slice (WK = 4: every wave forms the whole 32x32 tile over a quarter of each slice, and the four results are added in wave
// order at the end).
// An operand tile lies in LDS in the orientation of its memory:
//   k contiguous ("KM"): LDS [rows][BK + 4]; a lane reads 4 consecutive k at once (16 bytes), good for four MFMAs;
//   rows contiguous:     LDS [BK][rows + 8]; a lane reads one k row's element per MFMA, consecutive lanes consecutive banks.
// MFMA number 4 u + j of a slice contracts k = 8 u + j (lanes 0-31) and 8 u + 4 + j (lanes 32-63): the order of k inside a slice
// is free as long as both operands agree.  Both paddings make the reads conflict-free (16 rows of BK + 4 floats start in 16
// different bank groups; the two halves of a wave read k rows that are 4 (rows + 8) floats, i.e. 32 banks, apart).
// Bound by the matrix pipes (256 flop per cycle and CU: 157 TFLOP/s at 2.4 GHz) and by how evenly the tiles fill 256 CUs; see
// choose() for which tile is taken.
// Measured: 4096^3 1.11 ms (124 TFLOP/s) with 128 tiles; 1024 x 1152 x 768 28-31 us with 32 tiles, 34-37 with 64, 69 with 128;
// 8192 x 768 x 768 103 us with 64 tiles, 115 with 128; 256 x 192 x 128 5 us with 32 tiles, 8 with 64.  The plain fp32-arithmetic
// kernel that ran before reached 10-12 TFLOP/s (307 us on average where these take 40).
// Strides and bases that do not allow 16-byte loads go through the scalar loader (VEC = 0).
#include <algorithm>

#include "nn.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int ROWS, int KM, int VEC, int BK>
struct Loader {
  static constexpr int LD = KM ? BK + 4 : ROWS + 8;
  static constexpr int ELEMS = KM ? ROWS * LD : BK * LD;
  static constexpr int CHUNKS = ROWS * BK / 4 / 256;  // groups of 4 floats per thread
  static constexpr int CPR = KM ? BK / 4 : ROWS / 4;  // groups per stored row
  f32x4 reg[CHUNKS];
  const float *p[CHUNKS];  // this thread's groups in the next slice
  bool row_ok[CHUNKS];
  int kk, kstep;           // k of the first group inside a slice; KM: the same for all, otherwise kstep more for each
  int64_t step;            // floats from one slice to the next
  // base = first row of the panel (KM) or first column (otherwise), k0 = first k
  __device__ __forceinline__ void init(const float *base, int64_t ld, int rows_left_, int k0) {
    kk = KM ? (threadIdx.x % CPR) * 4 : threadIdx.x / CPR;
    kstep = KM ? 0 : 256 / CPR;
    step = KM ? BK : BK * ld;
    rows_left = rows_left_;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = threadIdx.x + 256 * i, major = c / CPR, minor = (c % CPR) * 4;
      const int r = KM ? major : minor, k = k0 + (KM ? minor : major);
      p[i] = KM ? base + r * ld + k : base + k * ld + r;
      row_ok[i] = r < rows_left;
    }
  }
  int rows_left;
  // the slice's groups into registers; k_left = k from the slice's first to the end of the contraction
  __device__ __forceinline__ void load(int k_left) {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int k = kk + i * kstep;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {
        // an aligned group that straddles the operand's edge holds at least one of its elements, so reading it is safe; elements
        // beyond the last k are dropped, rows beyond the last give results that are not stored
        if (row_ok[i] && k < k_left) v = *reinterpret_cast<const f32x4 *>(p[i]);
        if (KM && k_left < BK) {
#pragma unroll
          for (int e = 1; e < 4; ++e) v[e] = k + e < k_left ? v[e] : 0.f;
        }
      } else {
        const int r = ((threadIdx.x + 256 * i) % CPR) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (KM ? (row_ok[i] && k + e < k_left) : (r + e < rows_left && k < k_left)) v[e] = p[i][e];
      }
      reg[i] = v;
      p[i] += step;
    }
  }
  __device__ __forceinline__ void store(float *lds) const {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = threadIdx.x + 256 * i;
      *reinterpret_cast<f32x4 *>(lds + (c / CPR) * LD + (c % CPR) * 4) = reg[i];
    }
  }
  // the lane's values for MFMAs 4 u .. 4 u + 3 of the 32 rows starting at row0
  static __device__ __forceinline__ f32x4 frag(const float *lds, int row0, int u) {
    const int c = threadIdx.x & 31, k = 8 * u + 4 * ((threadIdx.x >> 5) & 1);
    if (KM) return *reinterpret_cast<const f32x4 *>(lds + (row0 + c) * LD + k);
    const float *p = lds + k * LD + row0 + c;
    return f32x4{p[0], p[LD], p[2 * LD], p[3 * LD]};
  }
};

struct Ep32 {
  float alpha;
  const float *bias, *residual;
  float *out;
  int64_t ldc;
};

// Grid: x = tiles (dealt so that each of the 8 XCDs walks a contiguous range, in columns of 8 tile rows), y = parts of the
// contraction (kchunk long, a multiple of BK; part p writes its partial product to out + p M ldc).
template <int AKM, int BKM, int BM, int BN, int WK, int BK, int VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, Ep32 ep, int tiles_m,
                                                       int tiles_n, int kchunk) {
  constexpr int WM = WK == 1 ? 2 : 1, WN = WM, TM = BM / WM / 32, TN = BN / WN / 32, US = BK / 8 / WK;  // US: groups of 4 MFMAs per slice and wave
  static_assert(WM * WN * WK == 4 && (WK == 1 || (TM == 1 && TN == 1)), "four waves divide the tile or the slice");
  using LA = Loader<BM, AKM, VEC, BK>;
  using LB = Loader<BN, BKM, VEC, BK>;
  __shared__ __attribute__((aligned(16))) float As[2][LA::ELEMS];
  __shared__ __attribute__((aligned(16))) float Bs[2][LB::ELEMS];
  const int nb = tiles_m * tiles_n;
  int bid = blockIdx.x;
  if (nb % 8 == 0) bid = (bid % 8) * (nb / 8) + bid / 8;
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int m0 = (first_m + (bid % per_group) % gsize) * BM, n0 = ((bid % per_group) / gsize) * BN;
  const int kbeg = blockIdx.y * kchunk, kend = min(K, kbeg + kchunk);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = WK == 1 ? (wave >> 1) * (BM / 2) : 0, wn = WK == 1 ? (wave & 1) * (BN / 2) : 0, u0 = WK == 1 ? 0 : wave * US;
  const float *pa = AKM ? A + (int64_t)m0 * lda : A + m0, *pb = BKM ? B + (int64_t)n0 * ldb : B + n0;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  LA la;
  LB lb;
  la.init(pa, lda, M - m0, kbeg);
  lb.init(pb, ldb, N - n0, kbeg);
  la.load(kend - kbeg);
  lb.load(kend - kbeg);
  la.store(As[0]);
  lb.store(Bs[0]);
  __syncthreads();
  int cur = 0;
  for (int k0 = kbeg; k0 < kend; k0 += BK, cur ^= 1) {
    const bool more = k0 + BK < kend;
    if (more) {
      la.load(kend - k0 - BK);
      lb.load(kend - k0 - BK);
    }
    // fragments of group u + 1 are fetched while the MFMAs of group u run
    f32x4 af[2][TM], bf[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) af[0][i] = LA::frag(As[cur], wm + i * 32, u0);
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[0][j] = LB::frag(Bs[cur], wn + j * 32, u0);
#pragma unroll
    for (int u = 0; u < US; ++u) {
      if (u + 1 < US) {
#pragma unroll
        for (int i = 0; i < TM; ++i) af[(u + 1) & 1][i] = LA::frag(As[cur], wm + i * 32, u0 + u + 1);
#pragma unroll
        for (int j = 0; j < TN; ++j) bf[(u + 1) & 1][j] = LB::frag(Bs[cur], wn + j * 32, u0 + u + 1);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[u & 1][i][e], bf[u & 1][j][e], acc[i][j], 0, 0, 0);
    }
    if (more) {
      la.store(As[cur ^ 1]);
      lb.store(Bs[cur ^ 1]);
    }
    __syncthreads();
  }
  // accumulator register r of lane (g = lane / 32, c = lane % 32): row 8 (r / 4) + 4 g + r % 4, column c: a store instruction writes
  // two rows of 128 consecutive bytes
  float *out = ep.out + (int64_t)blockIdx.y * M * ep.ldc;
  auto put = [&](int m, int n, float x, float bias) {
    if (m >= M) return;
    float v = (x + bias) * ep.alpha;
    const int64_t o = (int64_t)m * ep.ldc + n;
    if (ep.residual) v += ep.residual[o];
    out[o] = v;
  };
  if (WK == 1) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn + 32 * j + (lane & 31);
      if (n >= N) continue;
      const float bias = ep.bias ? ep.bias[n] : 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) put(m0 + wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), n, acc[i][j][r], bias);
    }
  } else {
    // every wave finishes a quarter of the rows: registers 4 w .. 4 w + 3 of all four waves
    float *part = &As[0][0];
    static_assert(sizeof(As) >= 4 * 1024 * sizeof(float), "four 32x32 results fit the A stages");
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave * 1024 + r * 64 + lane] = acc[0][0][r];
    __syncthreads();
    const int n = n0 + (lane & 31);
    const float bias = ep.bias && n < N ? ep.bias[n] : 0.f;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int r = 4 * wave + rr;
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) x += part[w * 1024 + r * 64 + lane];
      if (n < N) put(m0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), n, x, bias);
    }
  }
}

template <int AKM, int BKM, int BM, int WK, int BK, int VEC>
void launch(hipStream_t st, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, const Ep32 &ep, int parts, int kchunk) {
  const int tm = (M + BM - 1) / BM, tn = (N + BM - 1) / BM;
  hipLaunchKernelGGL((gemm_f32_kernel<AKM, BKM, BM, BM, WK, BK, VEC>), dim3(tm * tn, parts), dim3(256), 0, st, M, N, K, A, lda, B, ldb, ep, tm, tn, kchunk);
}

template <int AKM, int BKM>
void launch_tile(hipStream_t st, int tile, bool vec, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, const Ep32 &ep, int parts,
                 int kchunk) {
  if (tile == 128 && vec) launch<AKM, BKM, 128, 1, 32, 1>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
  else if (tile == 128) launch<AKM, BKM, 128, 1, 32, 0>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
  else if (tile == 64 && vec) launch<AKM, BKM, 64, 1, 64, 1>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
  else if (tile == 64) launch<AKM, BKM, 64, 1, 64, 0>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
  else if (vec) launch<AKM, BKM, 32, 4, 64, 1>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
  else launch<AKM, BKM, 32, 4, 64, 0>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Tile and number of parts of the contraction, by estimated time: the busiest of 256 CUs works through ceil(tiles parts / 256)
// tiles at the share of the matrix peak that the tile reaches (measured over many rounds: 128 0.78, 64 0.6, 32 0.45; a quarter less
// where a CU holds one workgroup and nothing hides its waits); a cut contraction adds the pass over the partial products.
struct Choice { int tile, parts; };
Choice choose(int M, int N, int K, bool may_split, size_t split_floats) {
  static const struct { int tile; double rate; } kinds[] = {{128, 0.78}, {64, 0.6}, {32, 0.45}};
  Choice best{64, 1};
  double best_us = 1e30;
  for (const auto &k : kinds) {
    const double tiles = (double)((M + k.tile - 1) / k.tile) * ((N + k.tile - 1) / k.tile);
    for (int parts = 1; parts <= 16; parts *= 2) {
      if (parts > 1 && (!may_split || K / parts < 256 || (double)parts * M * N > (double)split_floats)) break;
      const double rounds = (double)(((int64_t)(tiles * parts) + 255) / 256);
      double us = rounds * 2.0 * k.tile * k.tile * K / parts / (0.61e6 * k.rate * (rounds == 1 ? 0.75 : 1.0));  // 0.61 TFLOP/s per CU
      if (parts > 1) us += 4.0 + (parts + 1.0) * M * N * 8.0 / 4e6;
      if (us < best_us) { best_us = us; best = {k.tile, parts}; }
    }
  }
  return best;
}

}  // namespace

void twist_gemm_f32_choice(const twist_ctx *ctx, int M, int N, int K, bool may_split, size_t split_floats, int &tile, int &parts, int &kchunk) {
  Choice ch = choose(M, N, K, may_split && !ctx->gemm_tile, split_floats);
  if (ctx->gemm_tile) ch = {ctx->gemm_tile == 128 ? 128 : 64, 1};
  const int bk = ch.tile == 128 ? 32 : 64;
  kchunk = ((K + ch.parts - 1) / ch.parts + bk - 1) / bk * bk;
  tile = ch.tile;
  parts = (K + kchunk - 1) / kchunk;
}

twist_status twist_gemm_f32(twist_ctx *ctx, hipStream_t st, GemmLayout lay, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                            int64_t ldc, const GemmEpilogue &e) {
  Ep32 ep{e.alpha, static_cast<const float *>(e.bias), e.residual, static_cast<float *>(e.out), ldc};
  const bool vec = aligned16(A) && aligned16(B) && lda % 4 == 0 && ldb % 4 == 0;
  int tile, parts, kchunk;
  twist_gemm_f32_choice(ctx, M, N, K, e.splitk_ws && !e.bias && !e.residual, e.splitk_floats, tile, parts, kchunk);
  if (parts > 1) ep = Ep32{1.f, nullptr, nullptr, e.splitk_ws, N};
  switch (lay) {
    case GEMM_NT: launch_tile<1, 1>(st, tile, vec, M, N, K, A, lda, B, ldb, ep, parts, kchunk); break;
    case GEMM_NN: launch_tile<1, 0>(st, tile, vec, M, N, K, A, lda, B, ldb, ep, parts, kchunk); break;
    case GEMM_TN: launch_tile<0, 0>(st, tile, vec, M, N, K, A, lda, B, ldb, ep, parts, kchunk); break;
  }
  TW_HIP(ctx, hipGetLastError());
  if (parts > 1) return twist_splitk_reduce(ctx, st, e.splitk_ws, parts, M, N, e.out, ldc, 1, e.alpha);
  return TWIST_OK;
}
