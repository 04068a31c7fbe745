// bf16 projections y = x W^T with both operands contiguous along the contraction: the ping-pong kernel of gemm.hip (256x256 or
// 256x128 workgroup tile, eight waves of 64x128 or 64x64 in two groups of four that run one phase apart) for that orientation.
//
// What bounded it: its loads fetched 64 bytes (32 k) of 16 rows each, half a cache line, at 570 ns per 32 KB and CU where whole lines
// come at 350; and v_mfma_f32_32x32x16_bf16 draws more power than 16x16x32 for the same product: on random operands a loop of
// nothing else runs at 1.76 against 2.04 PFLOP/s before the chip lowers its clock.  Hence
//  - the two 32-deep sub-tiles that share a row's 128-byte lines are fetched by consecutive instructions (400 ns per 32 KB), every
//    second sub-tile, three and four sub-tiles ahead: a ring of five stages, all of the CU's 160 KB;
//  - 16x16x32 products, B's fragment as first factor, so that a lane ends up with four adjacent columns of one row.
// Normally distributed operands, both kernels in one session: 8192^3 880 -> 810 us (1.36 PFLOP/s), 8192 x 6144 x 4096 333 -> 289,
// 8192 x 32000 x 2048 950 -> 858, 8192 x 5632 x 2048 166 -> 147.
// The same for an operand that is read back with the transposing LDS load gained nothing (its rows of 512 bytes are whole lines already
// and its memory phase is the longer one): those orientations stay in gemm.hip.
// LOSS: a vocabulary projection whose caller only wants the cross-entropy (evaluation).  A lane holds 4 columns of every 16 of a row, so
// a row's maximum and sum of exponentials over a wave's columns take two exchanges between lanes, and nothing but those two numbers is
// written: no burst of stores, no second pass.  4096 x 50257 x 768 with its loss: 397 + 76 us (logits written, read again) -> 337 + 6.
#include <algorithm>

#include "gemm_tile.h"

namespace {

constexpr int SK = 32, NST = 5;  // k extent of a sub-tile, stages
#define NT_WAIT(vm) __builtin_amdgcn_s_waitcnt(0x0070 | (vm))  // vmcnt(vm < 16), lgkmcnt(0)

// One operand: LDS [ROWS][4 chunks of 16 bytes]; chunk c of row r sits at position c ^ (-(r >> 2) & 3).  A fragment read takes chunk
// l / 16 of row l % 16, and the hardware serves lanes {0-3, 12-15, 20-23, 24-27} and so on together: these then lie in different banks.
__device__ __forceinline__ int swz(int r) { return -(r >> 2) & 3; }
template <int ROWS>
struct Loader {
  static constexpr int NP = ROWS / 128;  // one-KB pieces per wave and sub-tile
  desc_t desc;
  uint32_t off[NP];  // byte offset of the lane's chunk in sub-tile 0 (kOob: outside the operand)
  int kk;            // k of that chunk inside a sub-tile (the same in all pieces: rows 128 apart)
  __device__ __forceinline__ void init(const uint16_t *base, int64_t ld, int rows_left, int K, int wave, int lane) {
    desc = make_desc(base, (uint32_t)(panel_span(1, ld, min(rows_left, ROWS), rows_left, K) * 2));
    const int r0 = 16 * wave + (lane >> 2), c = (lane & 3) ^ swz(r0);
    kk = c * 8;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int r = r0 + 128 * i;
      off[i] = r < rows_left ? (uint32_t)((r * ld + kk) * 2) : kOob;
    }
  }
  // start the loads of sub-tiles u and u + 1 into the operand's parts of their stages at d0 and d1 (wave-uniform)
  __device__ __forceinline__ void issue_pair(int u, int K, const char *d0, const char *d1, int wave) const {
    const bool in0 = u * SK + kk < K, in1 = (u + 1) * SK + kk < K;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      dma16(desc, d0 + (wave + 8 * i) * 1024, in0 ? off[i] + u * (SK * 2) : kOob);
      dma16(desc, d1 + (wave + 8 * i) * 1024, in1 ? off[i] + (u + 1) * (SK * 2) : kOob);
    }
  }
};

template <int BN, bool LOSS>
__global__ __launch_bounds__(512) void gemm_nt_kernel(int M, int N, int K, const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, Ep ep, int tiles_m,
                                                      int tiles_n, const int32_t *targets, float *loss_parts, float *target_logit) {
  constexpr int TM = 4, TN = BN / 32, WN = BN / 2;  // 16x16 tiles of a wave, its columns
  constexpr int OPA = 256 * SK * 2, STG = OPA + BN * SK * 2;  // bytes of A's sub-tile; of a stage: A, then B
  constexpr int LPP = 4 + BN / 64;               // loads per pair of sub-tiles and wave
  constexpr int EPI_LD = WN + 4;                 // floats per staged output row: an odd number of 16-byte slots
  constexpr int LPR = WN / 4, RPI = 64 / LPR;    // lanes per output row, rows per store instruction
  static_assert(8 * 32 * EPI_LD * 4 <= NST * STG, "the results are turned through the stages");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STG];
  const int nb = tiles_m * tiles_n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wpos = wave & 3, half = wave >> 2;  // waves w and w+4 share a SIMD and sit in different groups
  const int wm = (wpos >> 1) * 128 + half * 64, wn = (wpos & 1) * WN;
  // fragment of 16 rows: lane l holds row l % 16, k = 8 (l / 16) .. + 7
  const int s = lane & 15, q = lane >> 4;
  const uint32_t fa = (uint32_t)((wm + s) * 64 + ((q ^ swz(s)) * 16)), fb = (uint32_t)(OPA + (wn + s) * 64 + ((q ^ swz(s)) * 16));
  // Persistent workgroups: each walks the tiles vid, vid + gridDim.x, ...  Tile numbers are dealt so that each of the 8 XCDs (own L2;
  // workgroup b runs on XCD b % 8) works on a contiguous range of tiles.
  for (int vid = blockIdx.x; vid < nb; vid += gridDim.x) {
  const int bid = nb % 8 == 0 ? (vid % 8) * (nb / 8) + vid / 8 : vid;
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int m0 = (first_m + (bid % per_group) % gsize) * 256, n0 = (bid % per_group) / gsize * BN;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  Loader<256> la;
  Loader<BN> lb;
  la.init(A + (int64_t)m0 * lda, lda, M - m0, K, wave, lane);
  lb.init(B + (int64_t)n0 * ldb, ldb, N - n0, K, wave, lane);
#pragma unroll
  for (int u = 0; u < 4; u += 2) {
    la.issue_pair(u, K, smem + u * STG, smem + (u + 1) * STG, wave);
    lb.issue_pair(u, K, smem + u * STG + OPA, smem + (u + 1) * STG + OPA, wave);
  }
  NT_WAIT(LPP);  // sub-tiles 0 and 1 have landed
  __builtin_amdgcn_s_barrier();
  if (half) __builtin_amdgcn_s_barrier();  // the second group runs one phase late
  const int nsub = (K + SK - 1) / SK;
  const char *cur = smem;  // stage of the sub-tile at work
  auto after = [&](const char *st, int n) { return st + (st + n * STG >= smem + NST * STG ? n - NST : n) * STG; };
  for (int u0 = 0; u0 < nsub; u0 += 2) {
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) {
      __builtin_amdgcn_sched_barrier(0);
      // memory phase: fragments of sub-tile u0 + odd; in every second one the loads of the two sub-tiles three and four ahead, into
      // the stages that both groups have left (beyond the last sub-tile the loads are out of range and just zero-fill)
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8 *>(cur + fa + i * 1024);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[j] = *reinterpret_cast<const bf16x8 *>(cur + fb + j * 1024);
      if (odd) {
        const char *d0 = after(cur, 3), *d1 = after(cur, 4);
        la.issue_pair(u0 + 4, K, d0, d1, wave);
        lb.issue_pair(u0 + 4, K, d0 + OPA, d1 + OPA, wave);
        NT_WAIT(LPP);  // own fragments are in registers; own loads of the next two sub-tiles have landed
      } else {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): own fragments are in registers
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      // compute phase; the columns are walked back and forth: one operand stays the same from each instruction to the next
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jj = 0; jj < TN; ++jj) {
          const int j = i & 1 ? TN - 1 - jj : jj;
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      cur = after(cur, 1);
    }
  }
  if (!half) __builtin_amdgcn_s_barrier();
  NT_WAIT(0);                    // own zero-filling loads beyond the last sub-tile
  __builtin_amdgcn_s_barrier();  // ... and everybody else's: LDS is reused below

  if constexpr (LOSS) {
    const int col0 = n0 + wn + 4 * q, blocks = 2 * tiles_n, block = col0 / WN;
    const bool edge = n0 + BN > N;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = m0 + wm + 16 * i + s;
      const int at = (row < M ? targets[row] : -1) - col0;  // the target's distance from the lane's first column
      float mx = -INFINITY, target = 0.f;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const uint32_t lo = pack_bf16(acc[i][j][0], acc[i][j][1]), hi = pack_bf16(acc[i][j][2], acc[i][j][3]);  // the logits as they would be stored
        acc[i][j] = f32x4{bf2f((uint16_t)lo), bf2f((uint16_t)(lo >> 16)), bf2f((uint16_t)hi), bf2f((uint16_t)(hi >> 16))};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (at == 16 * j + e) target = acc[i][j][e];
          if (edge && col0 + 16 * j + e >= N) acc[i][j][e] = -INFINITY;
          mx = fmaxf(mx, acc[i][j][e]);
        }
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float ref = mx == -INFINITY ? 0.f : mx;
      float sum = 0.f;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += __expf(acc[i][j][e] - ref);
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      if (row >= M) continue;
      if (q == 0) *reinterpret_cast<f32x2 *>(loss_parts + ((int64_t)row * blocks + block) * 2) = f32x2{mx, sum};
      if (at >= 0 && at < WN && (at & 15) < 4) target_logit[row] = target;
    }
    continue;
  }
  // Epilogue.  Of a 16x16 accumulator tile a lane holds columns 4 (lane / 16) .. + 3 of row lane % 16; each wave turns its results
  // through LDS, 32 rows at a time, so that a store instruction writes two full rows of 128 columns (four of 64).
  float *stage = reinterpret_cast<float *>(smem + wave * (32 * EPI_LD * 4));
  const int cq = lane % LPR, rq = lane / LPR;
  float *const put = stage + s * EPI_LD + 4 * q;
  const int ncol = n0 + wn + 4 * cq;  // first of this lane's 4 columns
  float bias[4] = {0.f, 0.f, 0.f, 0.f};
  if (ep.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (ncol + e < N) bias[e] = bf2f(static_cast<const uint16_t *>(ep.bias)[ncol + e]);
  }
  const bool vec = ep.vec_ok && ncol + 3 < N;
  // a tile that lies inside the output and needs nothing but the conversion (most projections): no edge tests, no arithmetic
  const bool bare = ep.vec_ok && !ep.act_out && !ep.bias && !ep.residual && ep.alpha == 1.f && m0 + 256 <= M && n0 + BN <= N;
#pragma unroll
  for (int i = 0; i < TM / 2; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4 *>(put + 16 * h * EPI_LD + 16 * j) = acc[2 * i + h][j];
    if (bare) {
      const int64_t o0 = (int64_t)(m0 + wm + 32 * i + rq) * ep.ldc + ncol;
#pragma unroll
      for (int p = 0; p < 32 / RPI; ++p) {
        const f32x4 v4 = *reinterpret_cast<const f32x4 *>(stage + (RPI * p + rq) * EPI_LD + 4 * cq);
        const int64_t o = o0 + RPI * p * ep.ldc;
        if (ep.out_f32) {
          __builtin_nontemporal_store(v4, reinterpret_cast<f32x4 *>(static_cast<float *>(ep.out) + o));
        } else {
          const u32x2 w = {pack_bf16(v4[0], v4[1]), pack_bf16(v4[2], v4[3])};
          __builtin_nontemporal_store(w, reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(ep.out) + o));
        }
      }
      continue;
    }
#pragma unroll 4
    for (int p = 0; p < 32 / RPI; ++p) {
      const int row = RPI * p + rq, m = m0 + wm + 32 * i + row;
      const f32x4 v4 = *reinterpret_cast<const f32x4 *>(stage + row * EPI_LD + 4 * cq);
      if (m < M && ncol < N) store_quad<true, true>(ep, ep.out, m, ncol, N, v4, bias, vec);
    }
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's staged results are in registers
  __builtin_amdgcn_s_barrier();        // everybody's are: the next tile's loads may overwrite the staging area
  }
}

}  // namespace

void twist_launch_gemm_nt(hipStream_t st, int bn, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const void *ep,
                          const int32_t *targets, float *loss_parts, float *target_logit) {
  const Ep &e = *static_cast<const Ep *>(ep);
  const int tm = (M + 255) / 256, tn = (N + bn - 1) / bn;
  const dim3 grid(std::min(tm * tn, 256)), block(512);
#define TW_NT(BN, LOSS) hipLaunchKernelGGL((gemm_nt_kernel<BN, LOSS>), grid, block, 0, st, M, N, K, a, lda, b, ldb, e, tm, tn, targets, loss_parts, target_logit)
  if (targets && bn == 256) TW_NT(256, true);
  else if (targets) TW_NT(128, true);
  else if (bn == 256) TW_NT(256, false);
  else TW_NT(128, false);
#undef TW_NT
}
