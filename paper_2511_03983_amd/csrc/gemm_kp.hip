// bf16 projections of middling size: workgroup tiles of 64 to 192 rows and columns, one for (almost) every CU, where tiles of 256 rows would
// leave CUs idle and tiles of 64x64 fetch everything many times.
//
// What bounds such a product is the path from the L2 into LDS (4096 x 768 x 2560 in 128x96 tiles, 1.15 MB to a CU: loads alone 19.2 of 20.7 us, products
// alone 11.1, fragment reads alone 11.0; 60 B/ns and CU over the whole launch, 71 from slice to slice), then LDS itself.  Hence
//  - the largest tile that still gives the CUs one each, and slices 64 deep, so that a row of a k-contiguous operand comes in whole lines;
//  - the two groups of four waves (one of each per SIMD) take every second slice of the whole tile instead of half the tile each: a
//    wave's part of the tile stays large (64x48 of 128x96), and a slice's fragments are read from LDS by four waves, not eight.  The
//    groups run one phase apart, as in gemm.hip: one reads its fragments while the other multiplies;
//  - the loads of the slice four ahead go into the stage a group has just left, spread between its products (issued in front of them:
//    2048 x 2048 x 768 13.1 us instead of 11.4; in the reading phase, one stage more: 4 % slower);
//  - the groups' sums meet in LDS at the end: each hands half of its rows over and finishes the other half.
// 64x96 takes 80 KB of LDS, so that two workgroups share a CU (six or eight stages, one workgroup: equal on 256 tiles, up to a third slower
// beyond).  Also measured: results stored straight from the registers (2-8 % slower); tiles of 64x128, 128x64, 64x192 and 64x64 of this
// build (with all of them in the rule another 0.3 % on average).  Of the fixed 6 us of a small product the kernel's own are 3: first
// loads 0.7, the sums' exchange 0.8, stores 0.7.
#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"

namespace {

constexpr int BK = 64;  // k extent of a slice: whole 128-byte lines of an operand that is contiguous along k
constexpr int NST = 4;  // stages

// One operand's slice: ROWS rows of the tile, BK deep, in the orientation of its memory; position p of a stored row holds chunk p ^ swz.
//   k contiguous (KM): [ROWS][8 chunks]; a fragment read takes chunk 4 ks + q of 16 rows for the lanes 16 q + s
//   rows contiguous:   [BK][ROWS / 8 chunks], read back with the transposing LDS load: two chunks of k rows 8 q .. 8 q + 3 per 16 lanes
template <int KM, int ROWS>
struct Slice {
  static constexpr int BYTES = ROWS * BK * 2, NP = BYTES / 4096;    // one-KB pieces per wave of a group
  static constexpr int LEN = (KM ? BK : ROWS) * 2, CPR = LEN / 16;  // bytes and chunks of a stored row
  static __device__ __forceinline__ int swz(int r) {
    if (KM) return (r >> 1) & 7;
    const int near = LEN % 256 == 0 ? 4 * (r & 3) : LEN % 128 == 0 ? 4 * ((r >> 1) & 1) : 0;  // four adjacent k rows (LEN = 192: apart by themselves)
    return near ^ 2 * ((r >> 3) & 1);                                                         // and those eight further
  }
  desc_t desc;
  uint32_t off[NP];  // byte offset of this lane's chunk in slice 0 (kOob: outside the operand)
  int kk[NP];        // k of that chunk inside a slice
  uint32_t kstep;    // bytes from one slice to the next
  // base = the tile's first row at the first k (KM), or the first k's row at the tile's first row
  __device__ __forceinline__ void init(const uint16_t *base, int64_t ld, int rows_left, int K, int wave, int lane) {
    desc = make_desc(base, (uint32_t)(panel_span(KM, ld, min(rows_left, ROWS), rows_left, K) * 2));
    kstep = KM ? BK * 2 : (uint32_t)(BK * ld * 2);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int id = 64 * (wave + 4 * i) + lane, r = id / CPR, c = (id % CPR) ^ swz(r);
      kk[i] = KM ? c * 8 : r;
      off[i] = (KM ? r : c * 8) < rows_left ? (uint32_t)((r * ld + c * 8) * 2) : kOob;
    }
  }
  // start the loads of piece i of slice u into the operand's part of its stage at dst (wave-uniform)
  __device__ __forceinline__ void issue(int i, int u, int K, char *dst, int wave) const {
    dma16(desc, dst + (wave + 4 * i) * 1024, u * BK + kk[i] < K ? off[i] + u * kstep : kOob);
  }
};

// Fragments (16 rows x 32 k: lane 16 q + s holds row s, k = 8 q .. 8 q + 7) of a slice for a wave whose rows start at row0
template <int KM, int ROWS, int NT>
struct Frags {
  using S = Slice<KM, ROWS>;
  uint32_t a[KM ? 2 : NT];
  __device__ __forceinline__ void init(int row0, int lane) {
    const int s = lane & 15, q = lane >> 4;
    if (KM) {
      a[0] = (uint32_t)((row0 + s) * S::LEN + ((q ^ S::swz(row0 + s)) << 4));  // (the same swizzle in all tiles: rows 16 apart)
      a[KM ? 1 : 0] = a[0] ^ 64u;
    } else {
#pragma unroll
      for (int i = 0; i < (KM ? 0 : NT); ++i) {
        const int k = 8 * q + (s >> 2), chunk = ((row0 + 16 * i) >> 3) + ((s >> 1) & 1);
        a[i] = (uint32_t)(k * S::LEN + ((chunk ^ S::swz(k)) << 4) + (s & 1) * 8);  // (the same swizzle 4 and 32 k rows further)
      }
    }
  }
  // tile i, k-step ks (32 wide)
  __device__ __forceinline__ bf16x8 get(const char *p, int i, int ks) const {
    if constexpr (KM) {
      return *reinterpret_cast<const bf16x8 *>(p + a[ks] + i * 16 * S::LEN);
    } else {
      typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
      const char *at = p + a[i] + ks * 32 * S::LEN;
      const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at));
      const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + 4 * S::LEN));
      const s16x8 v = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
      return __builtin_bit_cast(bf16x8, v);
    }
  }
};

#define KP_WAIT(vm) __builtin_amdgcn_s_waitcnt(0x0070 | ((vm) & 15) | ((vm) >> 4) << 14)  // vmcnt(vm < 64), lgkmcnt(0)
#define KP_WAIT_LGKM0 __builtin_amdgcn_s_waitcnt(0xc07f)                                 // lgkmcnt(0)
#define KP_WAIT_VM(vm) __builtin_amdgcn_s_waitcnt(0x0f70 | ((vm) & 15) | ((vm) >> 4) << 14)

// G: TnGroup for the tiles of several weight gradients in one launch, tiles_m in all (tiles_n = 1).  gridDim.y parts of the contraction.
template <int AKM, int BKM, int BM, int BN, class G = NoGroup>
__global__ __launch_bounds__(512) void gemm_kp_kernel(int M, int N, int K, const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, Ep ep, int tiles_m,
                                                      int tiles_n, int kchunk, G group) {
  using OA = Slice<AKM, BM>;
  using OB = Slice<BKM, BN>;
  constexpr int TM = BM / 32, TN = BN / 32;                          // 16x16 tiles of a wave: half the rows, half the columns
  constexpr int STG = OA::BYTES + OB::BYTES, LPS = OA::NP + OB::NP;  // bytes of a stage, loads per slice and wave
  constexpr int LDE = BN + 4;                                        // floats per row of results in LDS: an odd number of 16-byte slots
  static_assert(BM % 64 == 0 && BN % 32 == 0 && BM * LDE * 4 <= NST * STG && NST * STG <= 160 * 1024, "the results are turned through the stages");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STG];
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
  const int half = wave >> 2, w4 = wave & 3;  // waves w and w + 4 share a SIMD; group `half` takes slices half, half + 2, ...
  const int wm = (w4 >> 1) * (BM / 2), wn = (w4 & 1) * (BN / 2);

  OA la;
  OB lb;
  la.init(AKM ? A + (int64_t)m0 * lda + kbeg : A + (int64_t)kbeg * lda + m0, lda, M - m0, Kl, w4, lane);
  lb.init(BKM ? B + (int64_t)n0 * ldb + kbeg : B + (int64_t)kbeg * ldb + n0, ldb, N - n0, Kl, w4, lane);
  auto issue = [&](int u, int from, int to) {  // pieces from .. to - 1 of slice u
    char *dst = smem + (uint32_t)u % NST * STG;
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
      if (i < from || i >= to) continue;
      if (i < OA::NP) la.issue(i < OA::NP ? i : 0, u, Kl, dst, w4);
      else lb.issue(i < OA::NP ? 0 : i - OA::NP, u, Kl, dst + OA::BYTES, w4);
    }
  };
  // Slice p is read in phase p; in phase p + 1 its group starts slice p + NST, into the stage that its four waves have left.
  constexpr int FLY = (NST / 2 - 1) * LPS;  // own loads still in flight when the group's next slice has landed
#pragma unroll
  for (int u = 0; u < NST; u += 2) issue(u + half, 0, LPS);
  Frags<AKM, BM, TM> fa;
  Frags<BKM, BN, TN> fb;
  fa.init(wm, lane);
  fb.init(wn, lane);
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  KP_WAIT_VM(FLY);
  __builtin_amdgcn_s_barrier();
  if (half) __builtin_amdgcn_s_barrier();  // the second group runs one phase late
  const int nsl = (Kl + BK - 1) / BK;
  for (int u0 = 0; u0 < nsl; u0 += 2) {
    const int u = u0 + half;
    const char *sa = smem + (uint32_t)u % NST * STG, *sb = sa + OA::BYTES;
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[ks][i] = fa.get(sa, i, ks);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[ks][j] = fb.get(sb, j, ks);
    }
    KP_WAIT_LGKM0;  // own fragments are in registers
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        issue(u + NST, (ks * TM + i) * LPS / (2 * TM), (ks * TM + i + 1) * LPS / (2 * TM));  // beyond the last slice out of range: zeros
#pragma unroll
        for (int jj = 0; jj < TN; ++jj) {
          const int j = i & 1 ? TN - 1 - jj : jj;
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ks][j], af[ks][i], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    KP_WAIT_VM(FLY);  // this wave's loads of the group's next slice have landed
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
  }
  if (!half) __builtin_amdgcn_s_barrier();
  KP_WAIT(0);                    // own zero-filling loads beyond the last slice
  __builtin_amdgcn_s_barrier();  // ... and everybody else's: LDS is reused below

  // Each group hands half of its rows' partial sums to the other and adds the other's to its own half; then the tile lies in LDS in rows.
  const int s = lane & 15, q = lane >> 4;
  float *const tile = reinterpret_cast<float *>(smem);
  float *const put = tile + (wm + s) * LDE + wn + 4 * q;
  // (first: the 16-row tile from which the group keeps TM / 2 of them)
  auto give = [&](auto first) {
    constexpr int I = TM / 2 - decltype(first)::value;
#pragma unroll
    for (int i = I; i < I + TM / 2; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4 *>(put + 16 * i * LDE + 16 * j) = acc[i][j];
  };
  auto take = [&](auto first) {
    constexpr int I = decltype(first)::value;
#pragma unroll
    for (int i = I; i < I + TM / 2; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4 *>(put + 16 * i * LDE + 16 * j) += acc[i][j];
  };
  using Low = std::integral_constant<int, 0>;
  using High = std::integral_constant<int, TM / 2>;
  if (half) give(High());
  else give(Low());
  __syncthreads();
  if (half) take(High());
  else take(Low());
  __syncthreads();
  void *const outp = gridDim.y > 1 ? static_cast<void *>(static_cast<float *>(ep.out) + (int64_t)blockIdx.y * M * ep.ldc) : ep.out;
  constexpr int QPR = BN / 4;  // groups of four columns in a row
  // A weight gradient goes past the caches, as from the 256-row tiles: nothing reads it before the optimizer, and what the following kernels read stays
  // (us of a pass, 256x128 tiles / these, kept in the caches / past them: 708 tokens, 176 wide, vocabulary 32000 341.5 / 349.9 / 336.9; 512 tokens, 616 wide, ten
  // layers 2265 / 2284 / 2239).  Partial products are read next.
  const bool stream = !AKM && gridDim.y == 1;
  // a tile that lies inside the output and needs nothing but the conversion: no edge tests, no arithmetic
  if (ep.vec_ok && !ep.act_out && !ep.bias && !ep.residual && ep.alpha == 1.f && m0 + BM <= M && n0 + BN <= N) {
#pragma unroll
    for (int id0 = 0; id0 < BM * QPR; id0 += 512) {
      const int id = id0 + threadIdx.x, row = id / QPR, c4 = id % QPR * 4;
      const f32x4 v = *reinterpret_cast<const f32x4 *>(tile + row * LDE + c4);
      const int64_t o = (int64_t)(m0 + row) * ep.ldc + n0 + c4;
      if (!AKM && stream && ep.out_f32) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(static_cast<float *>(outp) + o));
      else if (ep.out_f32) *reinterpret_cast<f32x4 *>(static_cast<float *>(outp) + o) = v;
      else *reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(outp) + o) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    }
    return;
  }
#pragma unroll 2
  for (int id0 = 0; id0 < BM * QPR; id0 += 512) {
    const int id = id0 + threadIdx.x, row = id / QPR, c4 = id % QPR * 4, m = m0 + row, ncol = n0 + c4;
    if (m >= M || ncol >= N) continue;
    float bias[4] = {0.f, 0.f, 0.f, 0.f};
    if (ep.bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ncol + e < N) bias[e] = bf2f(static_cast<const uint16_t *>(ep.bias)[ncol + e]);
    }
    const f32x4 v = *reinterpret_cast<const f32x4 *>(tile + row * LDE + c4);
    const bool vec = ep.vec_ok && ncol + 3 < N;
    if (!AKM && stream) store_quad<true, false>(ep, outp, m, ncol, N, v, bias, vec);
    else store_quad<false, AKM && BKM>(ep, outp, m, ncol, N, v, bias, vec);
  }
}

template <int BM, int BN>
void launch(hipStream_t st, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const Ep &ep, int parts, int kchunk) {
  const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  const dim3 grid(tm * tn, parts), block(512);
  switch (lay) {
    case GEMM_NT: hipLaunchKernelGGL((gemm_kp_kernel<1, 1, BM, BN>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, kchunk, NoGroup()); break;
    case GEMM_NN: hipLaunchKernelGGL((gemm_kp_kernel<1, 0, BM, BN>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, kchunk, NoGroup()); break;
    case GEMM_TN: hipLaunchKernelGGL((gemm_kp_kernel<0, 0, BM, BN>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, kchunk, NoGroup()); break;
  }
}

}  // namespace

void twist_launch_gemm_kp(hipStream_t st, int bm, int bn, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb,
                          const void *ep, int parts, int kchunk) {
  const Ep &e = *static_cast<const Ep *>(ep);
  if (bm == 128 && bn == 192) launch<128, 192>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
  else if (bm == 192) launch<192, 128>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
  else if (bm == 128 && bn == 128) launch<128, 128>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
  else if (bm == 128) launch<128, 96>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
  else launch<64, 96>(st, lay, M, N, K, a, lda, b, ldb, e, parts, kchunk);
}

void twist_launch_gemm_kp_group(hipStream_t st, int bm, int bn, const void *group, int tiles, int K, const void *ep, int parts, int kchunk) {
  const Ep &e = *static_cast<const Ep *>(ep);
  const TnGroup &g = *static_cast<const TnGroup *>(group);
  const dim3 grid(tiles, parts), block(512);
#define TW_KP(BM, BN) hipLaunchKernelGGL((gemm_kp_kernel<0, 0, BM, BN, TnGroup>), grid, block, 0, st, 0, 0, K, nullptr, 0, nullptr, 0, e, tiles, 1, kchunk, g)
  if (bm == 128 && bn == 192) TW_KP(128, 192);
  else if (bm == 192) TW_KP(192, 128);
  else if (bm == 128 && bn == 128) TW_KP(128, 128);
  else if (bm == 128) TW_KP(128, 96);
  else TW_KP(64, 96);
#undef TW_KP
}
