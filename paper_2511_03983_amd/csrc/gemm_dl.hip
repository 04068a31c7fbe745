// bf16 projections with too few 256-row tiles to fill the chip: workgroup tiles of 64x64 and of 32x32.
//
// What bounds such a product is latency: the contraction is short (a few hundred to a few thousand), so a tile is a short chain of
// load - barrier - multiply steps between a launch and an epilogue, and what counts is how long the chain is and how much is
// in flight.  Both kernels fetch their operands with loads straight into LDS (lane l of a wave writes 16 bytes at base + 16 l), four
// stages of 16 KB; 64 KB of LDS per workgroup, so two of them share a CU and one's waits and epilogue run under the other's products.
//   64x64, slices of 64:   four waves of 32x32;
//   32x32, slices of 128:  every wave forms the whole tile over a quarter of each slice (WK = 4); the four results are added
//                          in wave order at the end.  Four times as many workgroups and half the chain, for few rows.
// Slices of 64 and up also mean that a row of a k-contiguous operand is read in whole 128-byte lines.  (128x128 tiles of the same
// build measured no better than 64x64 or the 256x128 ping-pong kernel at any size tried: with one barrier for everybody a slice's loads,
// LDS reads and products, 256 cycles each, hardly overlap.)
// The times of all kernels side by side are with the rule that chooses between them, in gemm.hip.
// An operand's slice lies in LDS in the orientation of its memory; since the lanes' write pattern is fixed, bank conflicts are
// avoided by permuting which 16-byte chunk a lane fetches (position p of a row holds chunk p ^ swz(row)):
//   k contiguous ("KM"): [rows][BK]; a fragment read takes the same chunk of 16 consecutive rows, 256 / (2 BK) of which share the
//                        banks' 256 bytes: swz spreads the others;
//   rows contiguous:     [BK][rows], read back with the transposing LDS load: four adjacent chunks of four consecutive k rows.
// The contraction may also be cut into gridDim.y parts (fp32 partial products, summed by twist_splitk_reduce).
#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"

namespace {

// One operand: ROWS rows of the tile, slices of BK
template <int KM, int ROWS, int BK>
struct Operand {
  static constexpr int BYTES = ROWS * BK * 2, NP = BYTES / 4096;      // one slice; one-KB pieces per wave
  static constexpr int LEN = (KM ? BK : ROWS) * 2, CPR = LEN / 16;    // bytes and chunks of a stored row
  static constexpr int RPP = 64 / CPR;                                // stored rows in a piece
  static __device__ __forceinline__ int swz(int r) {
    if (KM) return CPR == 4 ? (r >> 2) & 3 : CPR == 8 ? (r >> 1) & 7 : r & 15;
    return CPR == 4 ? 0 : CPR == 8 ? 4 * ((r >> 1) & 1) : 4 * (r & 3);
  }
  desc_t desc;
  uint32_t off[NP];  // byte offset of this lane's chunk in slice 0 (kOob: outside the operand)
  int kk[NP];        // k of that chunk inside a slice
  uint32_t kstep;    // bytes from one slice to the next
  // base = the tile's first row at the first k (KM), or the first k's row at the tile's first row
  __device__ __forceinline__ void init(const uint16_t *base, int64_t ld, int rows_left, int K, int wave, int lane) {
    const int64_t span = panel_span(KM, ld, min(rows_left, ROWS), rows_left, K);
    desc = make_desc(base, (uint32_t)(span * 2));
    kstep = KM ? BK * 2 : (uint32_t)(BK * ld * 2);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int r = RPP * (wave + 4 * i) + lane / CPR, c = (lane % CPR) ^ swz(r);
      const int row = KM ? r : c * 8;
      kk[i] = KM ? c * 8 : r;
      off[i] = row < rows_left ? (uint32_t)((KM ? r * ld + c * 8 : r * ld + c * 8) * 2) : kOob;
    }
  }
  __device__ __forceinline__ void issue(int u, int K, char *dst, int wave) const {
#pragma unroll
    for (int i = 0; i < NP; ++i) dma16(desc, dst + (wave + 4 * i) * 1024, u * BK + kk[i] < K ? off[i] + u * kstep : kOob);
  }
};

// Fragments (32 rows x 16 k) of an operand's slice for a wave whose rows start at row0 and whose k starts at k0
template <int KM, int ROWS, int BK, int NT>
struct Frags {
  using O = Operand<KM, ROWS, BK>;
  uint32_t base;           // KM: the lane's row
  uint32_t x;              // KM: its swizzle
  uint32_t a[KM ? 1 : NT]; // otherwise: byte offset of the lane's part of tile i
  int c0;
  __device__ __forceinline__ void init(int row0, int k0, int lane) {
    const int c = lane & 31, g = lane >> 5, s = lane & 15, hi = (lane >> 4) & 1;
    if (KM) {
      base = (uint32_t)((row0 + c) * O::LEN);
      x = (uint32_t)O::swz(row0 + c);  // the same for all tiles: rows 32 apart
      c0 = k0 / 8 + g;
    } else {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const int k = k0 + g * 8 + (s >> 2), chunk = ((row0 + 32 * i) >> 3) + 2 * hi + ((s >> 1) & 1);
        a[i] = (uint32_t)(k * O::LEN + ((chunk ^ O::swz(k)) << 4) + (s & 1) * 8);
      }
    }
  }
  // tile i, k-step ks (16 wide)
  __device__ __forceinline__ bf16x8 get(const char *p, int i, int ks) const {
    if (KM) return *reinterpret_cast<const bf16x8 *>(p + base + i * 32 * O::LEN + ((((uint32_t)(c0 + 2 * ks)) ^ x) << 4));
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const char *q = p + a[i] + ks * 16 * O::LEN;  // 16 k rows further: the same swizzle
    s16x4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q));
    s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q + 4 * O::LEN));  // 4 k rows further: likewise (CPR >= 8), or none
    s16x8 w = {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
    return __builtin_bit_cast(bf16x8, w);
  }
};

#define DL_WAIT(vm) __builtin_amdgcn_s_waitcnt(0x0070 | ((vm) & 15) | ((vm) >> 4) << 14)  // vmcnt(vm < 64), lgkmcnt(0)

// G: TnGroup for the tiles of several weight gradients in one launch, tiles_m in all (tiles_n = 1)
template <int AKM, int BKM, int BM, int BN, int BK, int WK, int NST, class G = NoGroup>
__global__ __launch_bounds__(256) void gemm_dl_kernel(int M, int N, int K, const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, Ep ep, int tiles_m,
                                                      int tiles_n, int kchunk, G group) {
  constexpr int WM = WK == 1 ? 2 : 1, TM = BM / WM / 32, TN = BN / WM / 32, KS = BK / 16 / WK;  // KS: k-steps per slice and wave
  using OA = Operand<AKM, BM, BK>;
  using OB = Operand<BKM, BN, BK>;
  constexpr int STG = OA::BYTES + OB::BYTES, LPS = OA::NP + OB::NP;  // bytes of a stage, loads per stage and wave
  constexpr int LDE = BN / WM + 8;                                    // floats per staged row of results
  constexpr int EPI = (WK == 1 ? 4 * 32 : 4 * BM) * LDE * 4;
  __shared__ __attribute__((aligned(1024))) char smem[NST * STG > EPI ? NST * STG : EPI];
  // workgroup b runs on XCD b % 8: every XCD (own L2) gets a contiguous range of tiles, walked in columns of 8 tile rows
  const int nb = tiles_m * tiles_n, xcd = blockIdx.x & 7, q8 = nb >> 3, r8 = nb & 7;
  int bid = xcd * q8 + min(xcd, r8) + (int)(blockIdx.x >> 3);
  if constexpr (std::is_same<G, TnGroup>::value) {
    const TnProduct &p = group.p[product_of(group, bid)];
    M = p.M; N = p.N; A = p.a; B = p.b; lda = p.lda; ldb = p.ldb; tiles_m = p.tiles_m; tiles_n = p.tiles_n;
    ep.out = p.out; ep.ldc = N; ep.alpha = p.alpha; ep.vec_ok = p.vec_ok;
  }
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int m0 = (first_m + (bid % per_group) % gsize) * BM, n0 = ((bid % per_group) / gsize) * BN;
  const int kbeg = blockIdx.y * kchunk, Kl = min(kchunk, K - kbeg);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = WK == 1 ? (wave >> 1) * (BM / 2) : 0, wn = WK == 1 ? (wave & 1) * (BN / 2) : 0;

  OA la;
  OB lb;
  la.init(AKM ? A + (int64_t)m0 * lda + kbeg : A + (int64_t)kbeg * lda + m0, lda, M - m0, Kl, wave, lane);
  lb.init(BKM ? B + (int64_t)n0 * ldb + kbeg : B + (int64_t)kbeg * ldb + n0, ldb, N - n0, Kl, wave, lane);
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    la.issue(u, Kl, smem + u * STG, wave);
    lb.issue(u, Kl, smem + u * STG + OA::BYTES, wave);
  }
  Frags<AKM, BM, BK, TM> fa;
  Frags<BKM, BN, BK, TN> fb;
  const int k0 = WK == 1 ? 0 : wave * (BK / WK);
  fa.init(wm, k0, lane);
  fb.init(wn, k0, lane);
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // While the products of slice u run, the fragments of slice u + 1 come from LDS and slices u + 2 .. u + NST from memory.
  const int nsub = (Kl + BK - 1) / BK;
  bf16x8 af[2][KS][TM], bfr[2][KS][TN];
  auto fetch = [&](int u, auto par) {
    constexpr int P = decltype(par)::value;
    const char *sa = smem + (u % NST) * STG, *sb = sa + OA::BYTES;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[P][ks][i] = fa.get(sa, i, ks);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[P][ks][j] = fb.get(sb, j, ks);
    }
  };
  auto step = [&](int u, auto par) {
    constexpr int P = decltype(par)::value;
    __builtin_amdgcn_sched_barrier(0);
    DL_WAIT((NST - 2) * LPS);      // this wave's loads of slice u + 1 have landed and its fragments of slice u are in registers
    __builtin_amdgcn_s_barrier();  // everybody's: slice u + 1 can be read, the stage of slice u be overwritten
    __builtin_amdgcn_sched_barrier(0);
    fetch(u + 1, std::integral_constant<int, P ^ 1>());
    char *dn = smem + (u % NST) * STG;  // beyond the last slice the loads are out of range and just fill zeros
    la.issue(u + NST, Kl, dn, wave);
    lb.issue(u + NST, Kl, dn + OA::BYTES, wave);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[P][ks][i], bfr[P][ks][j], acc[i][j], 0, 0, 0);
  };
  DL_WAIT((NST - 1) * LPS);
  __builtin_amdgcn_s_barrier();
  fetch(0, std::integral_constant<int, 0>());
  for (int u = 0; u < nsub; u += 2) {
    step(u, std::integral_constant<int, 0>());
    if (u + 1 < nsub) step(u + 1, std::integral_constant<int, 1>());
  }
  DL_WAIT(0);
  __builtin_amdgcn_s_barrier();  // the stages are free: the results are turned through them so that a lane owns 4 adjacent columns

  // a 32x32 accumulator tile holds column lane % 32 and rows 8 (r / 4) + 4 (lane / 32) + r % 4
  const int c = lane & 31, g = lane >> 5;
  void *const outp = gridDim.y > 1 ? static_cast<void *>(static_cast<float *>(ep.out) + (int64_t)blockIdx.y * M * ep.ldc) : ep.out;
  float *stage = reinterpret_cast<float *>(smem);
  constexpr int LPR = BN / WM / 4, RPI = 64 / LPR;  // lanes per stored row, rows per store instruction
  const int cq = lane % LPR, rq = lane / LPR, ncol = n0 + wn + 4 * cq;
  float bias[4] = {0.f, 0.f, 0.f, 0.f};
  if (ep.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (ncol + e < N) bias[e] = bf2f(static_cast<const uint16_t *>(ep.bias)[ncol + e]);
  }
  const bool vec = ep.vec_ok && ncol + 3 < N;
  if (WK == 1) {
    stage += wave * (32 * LDE);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) stage[(8 * (r >> 2) + 4 * g + (r & 3)) * LDE + 32 * j + c] = acc[i][j][r];
#pragma unroll 4
      for (int p = 0; p < 32 / RPI; ++p) {
        const int row = RPI * p + rq, m = m0 + wm + 32 * i + row;
        const f32x4 v4 = *reinterpret_cast<const f32x4 *>(stage + row * LDE + 4 * cq);
        if (m < M && ncol < N) store_quad<false, AKM && BKM>(ep, outp, m, ncol, N, v4, bias, vec);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) stage[(wave * BM + 32 * i + 8 * (r >> 2) + 4 * g + (r & 3)) * LDE + 32 * j + c] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < BM / 4 / RPI; ++p) {  // every wave finishes a quarter of the rows
      const int row = wave * (BM / 4) + RPI * p + rq, m = m0 + row;
      f32x4 v4 = *reinterpret_cast<const f32x4 *>(stage + row * LDE + 4 * cq);
#pragma unroll
      for (int w = 1; w < 4; ++w) v4 += *reinterpret_cast<const f32x4 *>(stage + (w * BM + row) * LDE + 4 * cq);
      if (m < M && ncol < N) store_quad<false, AKM && BKM>(ep, outp, m, ncol, N, v4, bias, vec);
    }
  }
}

template <int BM, int BK, int WK, int NST>
void launch(hipStream_t st, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const Ep &ep, int parts, int kchunk) {
  const int tm = (M + BM - 1) / BM, tn = (N + BM - 1) / BM;
  const dim3 grid(tm * tn, parts), block(256);
  switch (lay) {
    case GEMM_NT: hipLaunchKernelGGL((gemm_dl_kernel<1, 1, BM, BM, BK, WK, NST>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, kchunk, NoGroup()); break;
    case GEMM_NN: hipLaunchKernelGGL((gemm_dl_kernel<1, 0, BM, BM, BK, WK, NST>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, kchunk, NoGroup()); break;
    case GEMM_TN: hipLaunchKernelGGL((gemm_dl_kernel<0, 0, BM, BM, BK, WK, NST>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, kchunk, NoGroup()); break;
  }
}

}  // namespace

void twist_launch_gemm_dl(hipStream_t st, int tile, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const void *ep,
                          int parts, int kchunk) {
  const Ep &e = *static_cast<const Ep *>(ep);
  if (tile == 32) launch<32, 128, 4, 4>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
  else launch<64, 64, 1, 4>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
}

void twist_launch_gemm_dl_group(hipStream_t st, int tile, const void *group, int tiles, int K, const void *ep, int parts, int kchunk) {
  const Ep &e = *static_cast<const Ep *>(ep);
  const TnGroup &g = *static_cast<const TnGroup *>(group);
  const dim3 grid(tiles, parts), block(256);
  if (tile == 32) hipLaunchKernelGGL((gemm_dl_kernel<0, 0, 32, 32, 128, 4, 4, TnGroup>), grid, block, 0, st, 0, 0, K, nullptr, 0, nullptr, 0, e, tiles, 1, kchunk, g);
  else hipLaunchKernelGGL((gemm_dl_kernel<0, 0, 64, 64, 64, 1, 4, TnGroup>), grid, block, 0, st, 0, 0, K, nullptr, 0, nullptr, 0, e, tiles, 1, kchunk, g);
}
