// Dense projections of the subnet: C = epilogue(op(A) op(B)) with fp32 accumulation.
//  - bf16 operands: MFMA kernels fed by direct-to-LDS loads: ping-pong kernels with tiles of 256x256 and 256x128 (here; in
//    gemm_nt.hip where both operands are contiguous along k), and 64x64 and 32x32 tiles for products too small to fill the
//    chip with those (gemm_dl.hip); operands stay in LDS in their memory orientation, and those whose contraction index is the slow
//    axis in memory are read back with the transposing LDS load.
//    Products between the two run on tiles of 64 to 192 rows and columns (gemm_kp.hip).
//  - fp32 operands: gemm_f32.hip.
//  - anything else (unaligned bf16 shapes, fp32 contractions of a few elements): a plain tiled FMA kernel with arbitrary strides.
#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"

namespace {

template <int BF>
__device__ __forceinline__ void store_out(const Ep &ep, int m, int n, float acc) {
  float v = acc;
  if (ep.bias) v += BF ? bf2f(static_cast<const uint16_t *>(ep.bias)[n]) : static_cast<const float *>(ep.bias)[n];
  v *= ep.alpha;
  const int64_t i = (int64_t)m * ep.ldc + n;
  if (ep.residual) v += ep.residual[i];
  if (ep.out_f32) static_cast<float *>(ep.out)[i] = v;
  else if (BF) static_cast<uint16_t *>(ep.out)[i] = f2bf(v);
  else static_cast<float *>(ep.out)[i] = v;
}

// ------------------------------------------------------------------------------------------- plain kernel
template <int BF>
__global__ __launch_bounds__(256) void gemm_plain_kernel(int M, int N, int K, const void *A, int64_t sam, int64_t sak, const void *B, int64_t sbk,
                                                         int64_t sbn, Ep ep) {
  __shared__ float As[16][65], Bs[16][65];
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4] = {};
  auto ld = [](const void *p, int64_t i) -> float {
    return BF ? bf2f(static_cast<const uint16_t *>(p)[i]) : static_cast<const float *>(p)[i];
  };
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int i = threadIdx.x; i < 1024; i += 256) {
      int r = i >> 4, k = i & 15;
      As[k][r] = (m0 + r < M && k0 + k < K) ? ld(A, (int64_t)(m0 + r) * sam + (int64_t)(k0 + k) * sak) : 0.f;
      Bs[k][r] = (n0 + r < N && k0 + k < K) ? ld(B, (int64_t)(k0 + k) * sbk + (int64_t)(n0 + r) * sbn) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = As[k][ty * 4 + i]; b[i] = Bs[k][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) {
      int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      if (m < M && n < N) store_out<BF>(ep, m, n, acc[i][j]);
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

// ------------------------------------------------------------------------------- ping-pong MFMA kernel
// 256x256 workgroup tile, 8 waves of 64x128, k walked in sub-tiles of 32.  The eight waves form two groups of
// four (one wave of each group per SIMD) that run the same loop one phase apart: while one group issues the
// 16 MFMAs of a sub-tile, the other reads its fragments of the next sub-tile from LDS and starts the global
// loads three sub-tiles ahead, so the matrix pipe of every SIMD always has a wave feeding it.
// Global loads go straight to LDS (buffer_load_dwordx4 ... lds: lane l of a wave writes 16 bytes at
// base + 16 l), four stages of 32 KB.  Because that write pattern is fixed, bank conflicts are avoided by
// permuting which 16-byte chunk of a row each lane fetches (an XOR swizzle) instead of by padding:
//   k contiguous in memory:    LDS [256 rows][4 chunks];  chunk c of row r sits at position c ^ ((r >> 2) & 3)
//   rows contiguous in memory: LDS [32 k][32 chunks];     chunk c of k-row k sits at position c ^ (4 (k & 3))
namespace pp {

constexpr int SK = 32;             // k extent of a sub-tile
constexpr int NST = 4;
#define PP_WAIT_VM_LGKM0(vm) __builtin_amdgcn_s_waitcnt(0x0070 | (vm))  // vmcnt(vm < 16) lgkmcnt(0)
#define PP_WAIT_VM0 __builtin_amdgcn_s_waitcnt(0x0f70)        // vmcnt(0)

template <int KM, int ROWS>
struct Loader {
  static constexpr int NP = ROWS / 128;  // one-KB pieces per wave
  static constexpr int CPR = ROWS / 8;   // rows contiguous: 16-byte chunks of a k row
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off[NP];  // byte offset of the lane's chunk in sub-tile 0 (kOob: outside the operand)
  int kk[NP];        // k of that chunk inside a sub-tile
  uint32_t kstep;   // bytes from one sub-tile to the next
  __device__ __forceinline__ void init(const uint16_t *base, int64_t ld, int rows_left, int K, int wave, int lane) {
    const int64_t span = panel_span(KM, ld, min(rows_left, ROWS), rows_left, K);
    rsrc = make_rsrc(base, (uint32_t)(span * 2));
    kstep = KM ? SK * 2 : (uint32_t)(SK * ld * 2);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int j = wave + 8 * i;  // which of the one-KB pieces of the sub-tile
      if (KM) {
        const int r = 16 * j + (lane >> 2), c = (lane & 3) ^ ((r >> 2) & 3);
        kk[i] = c * 8;
        off[i] = r < rows_left ? (uint32_t)((r * ld + c * 8) * 2) : kOob;
      } else {
        const int k = 64 / CPR * j + lane / CPR, c = (lane % CPR) ^ (4 * (k & 3));
        kk[i] = k;
        off[i] = c * 8 < rows_left ? (uint32_t)((k * ld + c * 8) * 2) : kOob;
      }
    }
  }
  // start the loads of sub-tile u into the operand's 16 KB at dst (wave-uniform)
  __device__ __forceinline__ void issue(int u, int K, char *dst, int wave) const {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const uint32_t o = (u * SK + kk[i] < K) ? off[i] + u * kstep : kOob;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void)(dst + (wave + 8 * i) * 1024), 16, o, 0, 0, 0);
    }
  }
};

// Per-lane LDS byte offsets (inside an operand's sub-tile) of the fragment reads of a wave whose rows start at wb.
template <int KM, int NTILE, int ROWS>
struct Frags {
  static constexpr int LEN = ROWS * 2;  // rows contiguous: bytes of a k row
  uint32_t a[KM ? 2 : NTILE];
  __device__ __forceinline__ void init(int wb, int lane) {
    const int c = lane & 31, g = lane >> 5, s = lane & 15, hi = (lane >> 4) & 1;
    if (KM) {
      a[0] = (uint32_t)((wb + c) * 64 + ((g ^ ((c >> 2) & 3)) * 16));
      a[1] = a[0] ^ 32u;
    } else {
#pragma unroll
      for (int i = 0; i < NTILE; ++i) {
        const int chunk = (wb >> 3) + 4 * i + 2 * hi + ((s >> 1) & 1);
        a[i] = (uint32_t)((g * 8 + (s >> 2)) * LEN + ((chunk ^ (4 * ((s >> 2) & 3))) * 16) + (s & 1) * 8);
      }
    }
  }
  // fragment of tile i (32 rows), k-step ks (16 wide) from the operand sub-tile at p
  __device__ __forceinline__ bf16x8 get(const char *p, int i, int ks) const {
    if (KM) return *reinterpret_cast<const bf16x8 *>(p + a[ks] + i * 2048);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const char *q = p + a[i] + ks * 16 * LEN;
    s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q));
    s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q + 4 * LEN));
    s16x8 v = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
};

// SPLIT: the k range is cut into `ksplit` parts of `kchunk` (a multiple of 32) and a work item is (part, tile); part p
// writes its unscaled fp32 partial product to ep.out + p * M * ldc and splitk_reduce_kernel adds the parts.  Used for
// products with few output tiles and a long k (weight gradients), which would otherwise occupy a fraction of the CUs.
// BN = 256, or 128: half as wide, 64x64 per wave, for products with too few tiles of 256.
// GROUP: the tiles of several weight gradients in one launch (with SPLIT; ksplit may be 1), nb tiles in all; their own sizes, operands
// and output replace the arguments'.
template <int AKM, bool SPLIT, int BN, class G = NoGroup>
__global__ __launch_bounds__(512) void gemm_pp_kernel(int M, int N, int K, const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, Ep ep,
                                                      int tiles_m, int tiles_n, int ksplit, int kchunk, G group) {
  constexpr bool GROUP_OF = std::is_same<G, TnGroup>::value;
  constexpr int TM = 2, TN = BN / 64, WN = BN / 2;
  constexpr int OPA = 256 * SK * 2, OPB = BN * SK * 2, STG = OPA + OPB;  // bytes of the operands' sub-tiles; one stage: A, then B
  constexpr int LPS = 2 + BN / 128;              // loads per sub-tile and wave
  constexpr int EPI_LD = WN + 8;                 // floats per staged output row: 4 rows apart = 32 banks apart
  constexpr int EPI_WAVE = 32 * EPI_LD * 4;      // one wave's 32 x WN block of fp32 results
  constexpr int LPR = WN / 4, RPI = 64 / LPR;    // lanes per output row, rows per store instruction
  constexpr int SMEM = NST * STG > 8 * EPI_WAVE ? NST * STG : 8 * EPI_WAVE;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  const int nb = GROUP_OF ? tiles_m : tiles_m * tiles_n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wpos = wave & 3, half = wave >> 2;  // waves w and w+4 share a SIMD and sit in different groups
  const int wm = (wpos >> 1) * 128 + half * 64, wn = (wpos & 1) * WN;
  Frags<AKM, TM, 256> fa;
  Frags<0, TN, BN> fb;
  fa.init(wm, lane);
  fb.init(wn, lane);
  // Persistent workgroups: each walks the tiles vid, vid + gridDim.x, ...; the stores of one tile drain while the
  // next tile's loads are already under way.  Tile numbers are dealt so that each of the 8 XCDs (own L2; workgroup
  // b runs on XCD b % 8) works on a contiguous range of tiles.
  const int n_items = SPLIT ? nb * ksplit : nb;
  for (int vid = blockIdx.x; vid < n_items; vid += gridDim.x) {
  int item = vid;
  if constexpr (GROUP_OF) item = (vid & 7) * (n_items >> 3) + min(vid & 7, n_items & 7) + (vid >> 3);  // an XCD's range stays within a part's k
  const int part = SPLIT ? item / nb : 0;
  int bid = SPLIT ? item - part * nb : item;
  if constexpr (GROUP_OF) {
    const TnProduct &p = group.p[product_of(group, bid)];
    M = p.M; N = p.N; A = p.a; B = p.b; lda = p.lda; ldb = p.ldb; tiles_m = p.tiles_m; tiles_n = p.tiles_n;
    ep.out = p.out; ep.ldc = N; ep.alpha = p.alpha; ep.vec_ok = p.vec_ok;
  } else if (nb % 8 == 0) {
    bid = (bid % 8) * (nb / 8) + bid / 8;
  }
  const int kbeg = SPLIT ? part * kchunk : 0;
  const int Kl = SPLIT ? min(kchunk, K - kbeg) : K;  // this item's k extent
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int tile_m = first_m + (bid % per_group) % gsize, tile_n = (bid % per_group) / gsize;
  const int m0 = tile_m * 256, n0 = tile_n * BN;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  Loader<AKM, 256> la;
  Loader<0, BN> lb;
  la.init(AKM ? A + (int64_t)m0 * lda + kbeg : A + (int64_t)kbeg * lda + m0, lda, M - m0, Kl, wave, lane);
  lb.init(B + (int64_t)kbeg * ldb + n0, ldb, N - n0, Kl, wave, lane);

  const int nsub = (Kl + SK - 1) / SK;
#pragma unroll
  for (int u = 0; u < NST - 1; ++u) {
    la.issue(u, Kl, smem + u * STG, wave);
    lb.issue(u, Kl, smem + u * STG + OPA, wave);
  }
  PP_WAIT_VM_LGKM0(2 * LPS);  // sub-tile 0 has landed
  __builtin_amdgcn_s_barrier();
  if (half) __builtin_amdgcn_s_barrier();  // the second group runs one phase late
  for (int u = 0; u < nsub; ++u) {
    const char *sa = smem + (u & (NST - 1)) * STG, *sb = sa + OPA;
    char *dn = smem + ((u + NST - 1) & (NST - 1)) * STG;
    __builtin_amdgcn_sched_barrier(0);
    // memory phase: fragments of sub-tile u; global loads of sub-tile u + 3 into the stage both groups left last
    // phase (beyond the last sub-tile the loads are out of range and just zero-fill)
    bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[ks][i] = fa.get(sa, i, ks);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[ks][j] = fb.get(sb, j, ks);
    }
    la.issue(u + NST - 1, Kl, dn, wave);
    lb.issue(u + NST - 1, Kl, dn + OPA, wave);
    PP_WAIT_VM_LGKM0(2 * LPS);  // own fragments are in registers; own loads of sub-tile u + 1 have landed
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // compute phase
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks][i], bfr[ks][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
  }
  if (!half) __builtin_amdgcn_s_barrier();
  PP_WAIT_VM0;                   // own zero-filling loads beyond the last sub-tile
  __builtin_amdgcn_s_barrier();  // ... and everybody else's: LDS is reused below

  // Epilogue.  A 32x32 accumulator tile holds column lane % 32 and rows 8*(r/4) + 4*(lane/32) + r%4, which
  // would store 2-byte pieces; each wave instead turns its results through LDS, 32 rows at a time, so that a
  // lane owns 4 consecutive columns and a store instruction writes two full rows of 128 columns (four of 64).
  float *stage = reinterpret_cast<float *>(smem + wave * EPI_WAVE);
  const int c = lane & 31, g = lane >> 5, cq = lane % LPR, rq = lane / LPR;
  void *const outp = SPLIT ? static_cast<void *>(static_cast<float *>(ep.out) + (int64_t)part * M * ep.ldc) : ep.out;
  const int ncol = n0 + wn + 4 * cq;  // first of this lane's 4 columns
  float bias[4] = {0.f, 0.f, 0.f, 0.f};
  if (ep.bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (ncol + e < N) bias[e] = bf2f(static_cast<const uint16_t *>(ep.bias)[ncol + e]);
  }
  const bool vec = ep.vec_ok && ncol + 3 < N;
  // a tile that lies inside the output and needs nothing but the conversion (most projections): no edge tests, no arithmetic
  const bool bare = ep.vec_ok && !ep.bias && !ep.residual && ep.alpha == 1.f && m0 + 256 <= M && n0 + BN <= N;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) stage[(8 * (r >> 2) + 4 * g + (r & 3)) * EPI_LD + 32 * j + c] = acc[i][j][r];
    if (bare) {
      const int64_t o0 = (int64_t)(m0 + wm + 32 * i + rq) * ep.ldc + ncol;
#pragma unroll
      for (int p = 0; p < 32 / RPI; ++p) {
        const f32x4 v4 = *reinterpret_cast<const f32x4 *>(stage + (RPI * p + rq) * EPI_LD + 4 * cq);
        const int64_t o = o0 + RPI * p * ep.ldc;
        if (ep.out_f32) {
          __builtin_nontemporal_store(v4, reinterpret_cast<f32x4 *>(static_cast<float *>(outp) + o));
        } else {
          const u32x2 w = {pack_bf16(v4[0], v4[1]), pack_bf16(v4[2], v4[3])};
          __builtin_nontemporal_store(w, reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(outp) + o));
        }
      }
      continue;
    }
#pragma unroll 4
    for (int p = 0; p < 32 / RPI; ++p) {
      const int row = RPI * p + rq, m = m0 + wm + 32 * i + row;
      const f32x4 v4 = *reinterpret_cast<const f32x4 *>(stage + row * EPI_LD + 4 * cq);
      if (m < M && ncol < N) store_quad<true, false>(ep, outp, m, ncol, N, v4, bias, vec);
    }
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's staged results are in registers
  __builtin_amdgcn_s_barrier();        // everybody's are: the next tile's loads may overwrite the staging area
  }
}

}  // namespace pp

// out = alpha * sum over parts of the fp32 partial products [parts][M][N] (parts added in ascending order)
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *ws, int parts, int M, int N, void *out, int64_t ldc, int out_f32, float alpha) {
  const int64_t total = (int64_t)M * N, i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= total) return;
  const bool vec = N % 4 == 0 && ldc % 4 == 0;  // then a group of 4 lies in one row and is 16-byte aligned
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < parts; ++p) {
    const float *src = ws + (int64_t)p * total + i;
    if (vec) {
      const f32x4 t = *reinterpret_cast<const f32x4 *>(src);
      v[0] += t[0]; v[1] += t[1]; v[2] += t[2]; v[3] += t[3];
    } else {
      for (int e = 0; e < 4 && i + e < total; ++e) v[e] += src[e];
    }
  }
  for (int e = 0; e < 4 && i + e < total; ++e) {
    const int64_t m = (i + e) / N, n = (i + e) - m * N, o = m * ldc + n;
    if (out_f32) static_cast<float *>(out)[o] = alpha * v[e];
    else static_cast<uint16_t *>(out)[o] = f2bf(alpha * v[e]);
  }
}

// the same for the products of a group, whose parts lie at p[].out; out[]: their gradients.  Blocks of 1024 elements, those of product i
// from first[i] on.
struct GroupOut { float *out[kGroupProducts]; int first[kGroupProducts]; };
__global__ __launch_bounds__(256) void group_reduce_kernel(TnGroup g, GroupOut o, int parts) {
  int q = 0;
#pragma unroll
  for (int i = 1; i < kGroupProducts; ++i)
    if (i < g.n && (int)blockIdx.x >= o.first[i]) q = i;
  const int64_t total = (int64_t)g.p[q].M * g.p[q].N, i = ((int64_t)(blockIdx.x - o.first[q]) * 256 + threadIdx.x) * 4;
  if (i >= total) return;
  const float *src = g.p[q].out + i;
  float *out = o.out[q] + i;
  if (total % 4 == 0 && ((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(src)) & 15) == 0) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int p = 0; p < parts; ++p) v += *reinterpret_cast<const f32x4 *>(src + p * total);
    *reinterpret_cast<f32x4 *>(out) = v * g.p[q].alpha;
  } else {
    for (int e = 0; e < 4 && i + e < total; ++e) {
      float v = 0.f;
      for (int p = 0; p < parts; ++p) v += src[p * total + e];
      out[e] = v * g.p[q].alpha;
    }
  }
}

// Measurement aid: nothing but the 32x32x16 matrix instruction of the kernels here (gemm_nt.hip uses 16x16x32), four independent accumulator tiles per wave
// (enough to issue back to back), operands in registers, no loads; the result is stored so that the loop stays.
// random_operands = 0: small constants (few bits toggle between instructions); 1: four different operand pairs of
// pseudo-random bf16 values of magnitude ~1 in rotation, which is what the multipliers see in a real projection and
// what the chip's power limit responds to.
__global__ __launch_bounds__(256) void mfma_only_kernel(int iters, float *sink, int random_operands) {
  bf16x8 a[4], b[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      uint32_t h = (threadIdx.x * 8u + i + 977u * j + 131071u * blockIdx.x) * 2654435761u;
      h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
      // sign and 7 mantissa bits at random, exponent in {2^-2 .. 2^1}: a spread like that of normalised activations
      const uint16_t ra = (uint16_t)(((h & 0x8000u)) | ((125u + ((h >> 7) & 3u)) << 7) | (h & 0x7fu));
      const uint16_t rb = (uint16_t)((((h >> 16) & 0x8000u)) | ((125u + ((h >> 23) & 3u)) << 7) | ((h >> 16) & 0x7fu));
      const uint16_t ca = (uint16_t)(0x3a80u + ((threadIdx.x + i) & 7)), cb = (uint16_t)(0x3b00u + ((threadIdx.x * 3 + i) & 7));
      a[j][i] = __builtin_bit_cast(__bf16, random_operands ? ra : ca);
      b[j][i] = __builtin_bit_cast(__bf16, random_operands ? rb : cb);
    }
  f32x16 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  for (int it = 0; it < iters; it += 4) {  // four iterations per trip so that the operand rotation is static
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j], b[(j + r) & 3], acc[j], 0, 0, 0);
  }
  float t = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) t += acc[j][r];
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = t;
}

// Which kernel a bf16 product runs on, and into how many parts its contraction is cut, by estimated time:
//   fixed + rounds * (tile + tile32 * (fp32 output) + slices * (s0 + s1 * share of the chip at work))   microseconds
// with slices of 32 along the contraction and rounds = how many tiles the busiest of 256 CUs works through.  fixed = launch; tile =
// first loads and epilogue of every tile, which decide where the contraction is short and the rows are many; s1 = how much slower a
// slice gets when the whole chip works (clock, memory); the 32x32 kernel's slices take nt of that where both operands are contiguous
// along k.  A cut contraction adds a launch and one pass over the fp32 partial products.
// Fitted to 800 products of every layout, sizes 1 to 50257, those of the TN layout cut in up to 16 parts (operands in rotation).  Over
// 300 others the kernel taken is on average 0.6 % slower than the fastest (without the cost of a tile, and with the rounds of the small
// tiles taken as items / 256, as the rule was: 2.7 %).  Some of them, us:
//   M x N x K             256x256  256x128   64x64   32x32
//   128 x 1536 x 2048        42.6     32.0     9.9     6.1
//   2048 x 2048 x 128        10.0      7.6     9.1    21.7
//   2048 x 1536 x 512        16.8     12.8    11.4    22.1   (fp32 output)
//   4096 x 768 x 2560        57.1     41.9    29.9    50.4   (fp32 output)
//   8192 x 768 x 64 (NN)      8.0      5.9    12.1    31.9
//   8192 x 768 x 192 (NN)    11.4     10.0    15.0    35.6   (fp32 output; the rule took 64x64 here)
//   8192 x 2048 x 256        15.6     17.4    32.9    81.8
//   8192 x 3072 x 1024 (NN)  56.9     60.5   108.6   228.3
//   8192 x 50257 x 64         340      465
//   1536 x 1536 x 2048 (TN)  39.5     33.8    25.3    47.5   (fp32 output)
// and cut: 768 x 640 x 4096 (TN) 17.5 whole, 15.2 in two parts, 17.5 in three; 2048 x 1024 x 8192 56 in five, 63 in eight;
// 256 x 128 x 2048 6.1 whole, 9.0 in eight.
struct Kind { int bm, bn; double fixed, tile, tile32, s0, s1, lay[3]; };  // lay: factors of a slice's time for GEMM_NT, NN, TN
constexpr Kind kKinds[] = {{256, 256, 1.0, 9.1, 0.36, 0.434, 0.32, {1, 1, 1}}, {256, 128, 1.7, 4.4, 1.0, 0.344, 0.23, {1, 1, 1}},
                           {64, 64, 2.95, 0.875, 0.19, 0.12, 0.011, {1, 1, 1}}, {32, 32, 2.5, 0.81, 0.06, 0.068, 0.01, {0.71, 1, 1}},
// Two groups that share the contraction (gemm_kp.hip).  Fitted to 600 products of their own, sizes 64 to 50257 (half of the estimates within
// 4 %, 8 % for 64x96; nine tenths within 13 and 18 %).  They are taken where they are expected to be a twelfth faster than the others (choose_any): of 200
// products not fitted to, 33 then went to them, 20 % faster on average and one slower, by 4.6 %; with the bare estimates 43, one of them
// 23 % slower.  Launches of fewer than 128 tiles (2048 x 896 x 3000, TN, 112 of 128x128: 22.8 us, 64x64 20.8), of fewer than 170 tiles of 96 columns, whose
// CUs have too little in flight where operands come from memory (37 products 4 % faster with operands in the caches, 8 % slower otherwise; 1536 x 1024 x
// 4096, NN, 132 tiles 26.2 / 28.0 and 29.9 / 36.4; 51 of 170 to 192 tiles 24 and 13 % faster), and of more than four rounds (50257 x 280 x 7007, TN: 383,
// 256x256 329) are left out, and contractions beyond 8192 (choose_any).  us, the others' fastest / these:
//   2816 x 2048 x 8192 (TN)      105 / 94   (192x128)      2048 x 768 x 2048 (f32)       15.3 / 11.8 (64x96)
//   4096 x 768 x 2560 (f32)     30.4 / 21.1 (128x96)       2048 x 1536 x 768             13.0 /  9.9 (128x96)
//   2048 x 2048 x 768           16.0 / 11.4 (128x128)      3000 x 2048 x 2488 (f32)      48.3 / 39.2 (192x128)
//   3000 x 2048 x 4976 (NN)     74.5 / 59.5 (192x128)      1024 x 2048 x 8192 (TN)       50.1 / 51.1 (128x128; 46 in two parts)
//   3072 x 2048 x 8192 (TN)      106 / 94   (192x128)
// and on the other side of the line 8192 x 768 x 768 16.2 / 15.2 (128x192), 8192 x 768 x 192 (NN, f32) 9.6 / 13.1, 4096 x 1920 x 768 16.5 / 19.1, 8192 x 1024 x 2048 33.2 / 35.0,
// 8192 x 5632 x 2048 144 / 200, 1024^3 7.2 / 7.9, 50257 x 768 x 8192 (TN) 594 / 732.
                           {128, 192, 1.62, 6.98, 0.31, 0.252, 0.118, {1, 1.045, 1.08}}, {192, 128, 1.09, 6.73, 0.33, 0.262, 0.1, {1, 1.005, 1.075}},
                           {128, 128, 1.98, 4.75, 0.34, 0.16, 0.09, {1, 1.01, 0.975}}, {128, 96, 2.66, 3.92, 0.35, 0.143, 0.058, {1, 1.105, 1.17}},
                           {64, 96, 5.52, 0.97, 0.3, 0.0865, 0.0335, {1, 1.085, 1.12}}};
constexpr int kOneGroup = 4, kAllKinds = sizeof(kKinds) / sizeof(kKinds[0]);  // kinds from kOneGroup on are those of gemm_kp.hip
struct Choice { int kind, parts; double us = 0.0, idle = 0.0; int64_t items = 0; };  // idle: of the microseconds, those of CUs without a tile
// parts of the contraction and their length, a multiple of the kernel's slices
struct Cut { int kind, parts, kchunk; };
Cut cut_into(int kind, int parts, int K) {
  const int step = kind < 2 ? 32 : 128, kchunk = ((K + parts - 1) / parts + step - 1) / step * step;
  return {kind, (K + kchunk - 1) / kchunk, kchunk};
}
// Of the k of a part those that one fp32 accumulator of a wave sums up.  The error of a product grows with the root of that number, whatever the
// instruction: 6728 x 136 x 7984 (TN) on 256x256 in nine parts 1.8e-7, on 64x96 whole 3.9e-7; uncut products of gemm_kp.hip are at 0.69 of the others.
double chain_of(int kind, int parts, int K) {
  const int k = std::min(K, cut_into(kind, parts, K).kchunk);
  return kind >= kOneGroup ? k / 2.0 : kind == 3 ? k / 4.0 : k;
}
// (several products over the same K that share a launch: their tiles and outputs together; among kinds first .. last - 1; sums no longer than `longest`)
Choice choose_of(int first, int last, GemmLayout lay, int n, const int *Ms, const int *Ns, int K, bool f32_out, int most_parts, size_t split_floats,
                 double longest = 1e30) {
  Choice best{first, 1, 1e30};
  double best_us = 1e30, outputs = 0.0;
  for (int i = 0; i < n; ++i) outputs += (double)Ms[i] * Ns[i];
  for (int k = first; k < last; ++k) {
    const Kind &kd = kKinds[k];
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (int64_t)((Ms[i] + kd.bm - 1) / kd.bm) * ((Ns[i] + kd.bn - 1) / kd.bn);
    for (int parts = 1; parts <= most_parts; ++parts) {
      if (parts > 1 && (K < 256 * parts || parts * outputs > (double)split_floats)) break;
      const int64_t items = tiles * parts, rounds = (items + 255) / 256;
      if (k >= kOneGroup && (items < (kd.bn == 96 ? 170 : 128) || items > 1024 || chain_of(k, parts, K) > longest)) continue;
      const double share = std::min(1.0, items / 256.0), slice = (kd.s0 + kd.s1 * share) * kd.lay[lay];
      double us = kd.fixed + rounds * (kd.tile + (f32_out || parts > 1 ? kd.tile32 : 0.0) + K / 32.0 / parts * slice);
      if (parts > 1) us += 4.4 + (parts + 1.0) * outputs * 4.0 / 2.8e6;
      if (us < best_us) { best_us = us; best = {k, parts, us, us * (1.0 - (k < 2 || k >= kOneGroup ? items / (256.0 * rounds) : share)), items}; }
    }
  }
  return best;
}
// the kernels whose waves share every slice
Choice choose(GemmLayout lay, int n, const int *Ms, const int *Ns, int K, bool f32_out, bool may_split, size_t split_floats) {
  return choose_of(0, kOneGroup, lay, n, Ms, Ns, K, f32_out, may_split ? 16 : 1, split_floats);
}
// all kernels.  Those of gemm_kp.hip cut a contraction no further than the others would, and sum no more coarsely.  Where it is as long as a vocabulary (its
// input gradient) they wait for memory: a CU has 120 KB in flight, and operands that come from beyond the caches take 2 us and more to arrive; us, the
// others / these: 8192 x 768 x 50257 778 / 741, 4096 x 512 x 50257 241 / 305, 1500 x 1024 x 32000 116 / 137, 8192 x 2048 x 32000 817 / 1074.  8192 is the longest
// they were fitted to, not where they cross: of longer ones some are faster (2816 x 2048 x 8200, TN, 121 / 108, 768 x 768 x 32768 78 / 66).
// Of the small tiles two share a CU, and their second round is shorter than the estimate has it (a tenth of the whole time): 0.82 there.  Tiles of 256x256
// suffer less from operands in memory: 11 products expected at 0.88 to 0.92 of their time took 0.99 with operands in the caches and 1.14 otherwise (8192 x 2304 x
// 768 43.5 / 40.1 and 42.9 / 49.8); 105 of 256x128 0.96 and 1.01.
Choice choose_any(GemmLayout lay, int n, const int *Ms, const int *Ns, int K, bool f32_out, bool may_split, size_t split_floats) {
  const Choice one = choose(lay, n, Ms, Ns, K, f32_out, may_split, split_floats);
  if (K > 8192) return one;
  const Choice two = choose_of(kOneGroup, kAllKinds, lay, n, Ms, Ns, K, f32_out, one.parts, split_floats, chain_of(one.kind, one.parts, K));
  return two.us < (one.kind >= 2 && one.items > 256 ? 0.82 : one.kind == 0 ? 0.88 : 0.92) * one.us ? two : one;
}

// kernel, parts of the contraction and their length of a bf16 product whose operands are aligned; `any`: among all kernels
Cut cut_of(const twist_ctx *ctx, bool any, GemmLayout lay, int M, int N, int K, bool f32_out, bool may_split, size_t split_floats) {
  Choice ch = (any ? choose_any : choose)(lay, 1, &M, &N, K, f32_out, may_split && lay != GEMM_NT, split_floats);
  if (ctx->gemm_tile) ch = {ctx->gemm_tile == 256 ? 0 : 1, 1};
  return cut_into(ch.kind, ch.parts, K);
}

// one launch of gemm_pp_kernel: kchunk = K for an uncut contraction, else a multiple of 32
template <int BN>
void launch_pp(hipStream_t st, GemmLayout lay, int M, int N, int K, const uint16_t *a, int64_t lda, const uint16_t *b, int64_t ldb, const Ep &ep, int parts, int kchunk) {
  const int tm = (M + 255) / 256, tn = (N + BN - 1) / BN;
  const dim3 grid(std::min(tm * tn * parts, 256)), block(512);
#define TW_PP(AKM)                                                                                                                                             \
  do {                                                                                                                                                              \
    if (parts > 1) hipLaunchKernelGGL((pp::gemm_pp_kernel<AKM, true, BN>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, parts, kchunk, NoGroup()); \
    else hipLaunchKernelGGL((pp::gemm_pp_kernel<AKM, false, BN>), grid, block, 0, st, M, N, K, a, lda, b, ldb, ep, tm, tn, 1, K, NoGroup());                   \
  } while (0)
  switch (lay) {
    case GEMM_NT: twist_launch_gemm_nt(st, BN, M, N, K, a, lda, b, ldb, &ep); break;  // never cut
    case GEMM_NN: TW_PP(1); break;
    case GEMM_TN: TW_PP(0); break;
  }
#undef TW_PP
}

// fp32 operands without padding have rows of whole 16-byte chunks
bool dense_rows_of_16(GemmLayout lay, int M, int N, int K) { return (lay == GEMM_TN ? M : K) % 4 == 0 && (lay == GEMM_NT ? K : N) % 4 == 0; }

// fp32 contractions within one slice of the plain kernel, with an output too large for the 32x32 tiles: bound by the stores, of which the
// plain kernel makes shorter work (us, plain / matrix instruction: 8192 x 2048 x 8 32 / 41, 512 x 50257 x 16 50 / 71, 3072 x 768 x 8 (TN)
// 9.9 / 13.8; from there on the other way: 8192 x 2048 x 32 40 / 38, 4096 x 4096 x 16 (TN) 41 / 37, 768 x 768 x 8 6.2 / 5.2).
bool short_f32(const twist_ctx *ctx, GemmLayout lay, int M, int N, int K) {
  if (K > (lay == GEMM_TN ? 8 : 16) || ctx->gemm_tile) return false;
  int tile, parts, kchunk;
  twist_gemm_f32_choice(ctx, lay, M, N, K, false, false, 0, tile, parts, kchunk);  // (measured against those kernels; K is a step of any)
  return tile > 32;
}

// twist_set_gemm_profile: events around a launch (the closing one on every return path) and its operations
struct GemmTimer {
  twist_ctx *ctx;
  hipStream_t st;
  hipEvent_t stop = nullptr;
  twist_status start(double flops) {
    if (!ctx->prof_gemm) return TWIST_OK;
    hipEvent_t begin, end;
    TW_HIP(ctx, hipEventCreate(&begin));
    TW_HIP(ctx, hipEventCreate(&end));
    ctx->prof_events.push_back(begin);
    ctx->prof_events.push_back(end);
    ctx->prof_flops += flops;
    TW_HIP(ctx, hipEventRecord(begin, st));
    stop = end;
    return TWIST_OK;
  }
  ~GemmTimer() { if (stop) (void)hipEventRecord(stop, st); }
};

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

twist_status twist_splitk_reduce(twist_ctx *ctx, hipStream_t st, const float *parts_ws, int parts, int M, int N, void *out, int64_t ldc, int out_f32, float alpha) {
  const int64_t groups = ((int64_t)M * N + 3) / 4;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st, parts_ws, parts, M, N, out, ldc, out_f32, alpha);
  TW_HIP(ctx, hipGetLastError());
  return TWIST_OK;
}

twist_status twist_gemm(twist_ctx *ctx, int bf16, GemmLayout lay, int M, int N, int K, const void *A, int64_t lda, const void *B, int64_t ldb,
                        int64_t ldc, const GemmEpilogue &e, hipStream_t st) {
  if (M <= 0 || N <= 0 || K <= 0) return TWIST_OK;
  const hipStream_t stream = st ? st : ctx->stream;
  if (e.act_out && (lay != GEMM_NT || ldc != N || stream != ctx->stream || (bf16 && e.out_f32) || (e.act != TWIST_ACT_GELU_TANH && e.act != TWIST_ACT_RELU)))
    TW_FAIL(ctx, TWIST_EINVAL, "projection: an ungated activation is applied to y = x W^T with unpadded rows in the model's type, on the context's stream only");
  GemmTimer timer{ctx, stream};
  TW_TRY(timer.start(2.0 * M * N * K));
  Ep ep{e.alpha, e.bias, e.residual, e.out, e.out_f32, ldc, nullptr, 0, 0};
  ep.vec_ok = ldc % 4 == 0 && aligned16(e.out) && (!e.residual || aligned16(e.residual)) && aligned16(e.act_out);
  const bool no_mfma = ctx->plain_only;
  // 16-byte chunks along k must not straddle the end of an operand row.  For y = x W with a ragged K the
  // caller pads x's rows (lda >= K rounded up to 8) with zeros; W's rows beyond K are never touched.
  const bool k_ok = lay == GEMM_TN || K % 8 == 0 || (lay == GEMM_NN && lda >= (K + 7) / 8 * 8);
  // buffer offsets are 32-bit: a row panel (256 rows) or a k-panel (K rows) of each operand and of C must stay below 2 GiB
  const int64_t a_span = (lay == GEMM_TN ? (int64_t)K : 256) * lda * 2, b_span = (lay == GEMM_NT ? 256 : (int64_t)K) * ldb * 2;
  const bool span_ok = a_span < (1ll << 31) && b_span < (1ll << 31) && 256 * ldc * 4 < (1ll << 31);
  const bool vec_ok = bf16 && !no_mfma && aligned16(A) && aligned16(B) && lda % 8 == 0 && ldb % 8 == 0 && k_ok && span_ok;
  if (vec_ok) {
    const uint16_t *a = static_cast<const uint16_t *>(A), *b = static_cast<const uint16_t *>(B);
    const Cut ch = cut_of(ctx, !e.targets, lay, M, N, K, e.out_f32, e.splitk_ws && !e.bias && !e.residual && aligned16(e.splitk_ws), e.splitk_floats);
    const int parts = ch.parts, kchunk = ch.kchunk;
    if (e.act_out) {
      ep.act_out = e.act_out;
      ep.act = e.act;
      if (e.act_only) ep.out = nullptr;
    }
    if (parts > 1) ep = Ep{1.f, nullptr, nullptr, e.splitk_ws, 1, N, nullptr, 0, N % 4 == 0};
    if (e.targets && lay == GEMM_NT && ch.kind < 2 && !e.out_f32 && !e.bias && !e.residual && e.alpha == 1.f) {
      twist_launch_gemm_nt(stream, ch.kind ? 128 : 256, M, N, K, a, lda, b, ldb, &ep, e.targets, e.loss_parts, e.target_logit);
      TW_HIP(ctx, hipGetLastError());
      *e.loss_blocks = 2 * ((N + kKinds[ch.kind].bn - 1) / kKinds[ch.kind].bn);
      return TWIST_OK;
    }
    switch (ch.kind) {
      case 0: launch_pp<256>(stream, lay, M, N, K, a, lda, b, ldb, ep, parts, kchunk); break;
      case 1: launch_pp<128>(stream, lay, M, N, K, a, lda, b, ldb, ep, parts, kchunk); break;
      case 2: twist_launch_gemm_dl(stream, 64, lay, M, N, K, a, lda, b, ldb, &ep, parts, kchunk); break;
      case 3: twist_launch_gemm_dl(stream, 32, lay, M, N, K, a, lda, b, ldb, &ep, parts, kchunk); break;
      default: twist_launch_gemm_kp(stream, kKinds[ch.kind].bm, kKinds[ch.kind].bn, lay, M, N, K, a, lda, b, ldb, &ep, parts, kchunk); break;
    }
    TW_HIP(ctx, hipGetLastError());
    return parts > 1 ? twist_splitk_reduce(ctx, stream, e.splitk_ws, parts, M, N, e.out, ldc, e.out_f32, e.alpha) : TWIST_OK;
  }
  auto activate = [&]() -> twist_status { return e.act_out ? twist_act_fwd(ctx, bf16, e.act, e.out, e.act_out, M, N) : TWIST_OK; };  // the kernels below do not
  if (!bf16 && !no_mfma && !short_f32(ctx, lay, M, N, K)) {
    TW_TRY(twist_gemm_f32(ctx, stream, lay, M, N, K, static_cast<const float *>(A), lda, static_cast<const float *>(B), ldb, ldc, e));
    return activate();
  }
  int64_t sam, sak, sbk, sbn;
  switch (lay) {
    case GEMM_NT: sam = lda; sak = 1; sbk = 1; sbn = ldb; break;
    case GEMM_NN: sam = lda; sak = 1; sbk = ldb; sbn = 1; break;
    default: sam = 1; sak = lda; sbk = ldb; sbn = 1; break;
  }
  dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
  if (bf16) hipLaunchKernelGGL(gemm_plain_kernel<1>, grid, block, 0, stream, M, N, K, A, sam, sak, B, sbk, sbn, ep);
  else hipLaunchKernelGGL(gemm_plain_kernel<0>, grid, block, 0, stream, M, N, K, A, sam, sak, B, sbk, sbn, ep);
  TW_HIP(ctx, hipGetLastError());
  return activate();
}

// What bound them: the weight gradients of one layer of a small model are too few tiles each to fill the chip, cut into many parts with
// a pass over the partial products behind each.  Together they fill it in fewer parts: 8192 x 768 x (192 heads, 768 hidden) in bf16 four
// launches and four sums, 109 us, against 45 + 6; 2048 x 768 x (512, 2048) 77 us against 44.  In fp32 (one stream, so where they are
// fewest): 256 x 128 x (64, 256) 20 us against 8, 1248 x 88 x (832, 344) 46 / 20, 1024 x 768 x (384, 1536) 98 / 63; of 156 such groups and pairs the
// mean is two thirds.
twist_status twist_weight_grads(twist_ctx *ctx, int bf16, int n, const WeightGrad *items, int K, float *scratch, size_t scratch_floats, hipStream_t st,
                                int32_t *chosen) {
  TnGroup g{};
  GroupOut o{};
  int Ms[kGroupProducts], Ns[kGroupProducts];
  // (fp32 contractions of a few elements: short_f32)
  bool one = !ctx->plain_only && !ctx->gemm_tile && n <= kGroupProducts && (bf16 || K > 8);
  for (int i = 0; i < n && one; ++i) {
    const WeightGrad &w = items[i];
    if (w.M <= 0 || w.N <= 0) continue;
    Ms[g.n] = w.M; Ns[g.n] = w.N;
    o.out[g.n] = w.out;
    g.p[g.n++] = {static_cast<const uint16_t *>(w.a), static_cast<const uint16_t *>(w.b), w.out, w.lda, w.ldb, w.M, w.N, 0, 0, 0, w.alpha, w.N % 4 == 0 && aligned16(w.out)};
    const int row = bf16 ? 8 : 4;  // elements that a row's stride is a multiple of
    one = aligned16(w.a) && aligned16(w.b) && w.lda % row == 0 && w.ldb % row == 0;
    if (bf16) one = one && K * w.lda * 2 < (1ll << 31) && K * w.ldb * 2 < (1ll << 31) && 256ll * w.N * 4 < (1ll << 31);
    else one = one && std::max(w.lda, w.ldb) < 1 << 23;
  }
  const bool may_split = scratch && aligned16(scratch);
  Cut ch{0, 1, K};
  int bm = 0, bn;
  one = one && g.n > 1 && K > 0;
  if (one && !bf16) one = twist_gemm_f32_group_choice(g.n, Ms, Ns, K, may_split ? scratch_floats : 0, bm, ch.parts, ch.kchunk);
  if (!one) {
    for (int i = 0; i < n; ++i) {
      GemmEpilogue e;
      e.alpha = items[i].alpha; e.out = items[i].out; e.out_f32 = 1;
      e.splitk_ws = scratch; e.splitk_floats = scratch_floats;
      TW_TRY(twist_gemm(ctx, bf16, GEMM_TN, items[i].M, items[i].N, K, items[i].a, items[i].lda, items[i].b, items[i].ldb, items[i].N, e, st));
    }
    return TWIST_OK;
  }
  const hipStream_t stream = st ? st : ctx->stream;
  GemmTimer timer{ctx, stream};
  double outputs = 0.0;
  for (int i = 0; i < g.n; ++i) outputs += (double)Ms[i] * Ns[i];
  TW_TRY(timer.start(2.0 * outputs * K));
  if (bf16) {
    const Choice c = choose_any(GEMM_TN, g.n, Ms, Ns, K, true, may_split, scratch_floats);
    ch = cut_into(c.kind, c.parts, K);
    bm = kKinds[ch.kind].bm;
    bn = kKinds[ch.kind].bn;
  } else {
    bn = bm;
  }
  if (chosen) { chosen[0] = bm; chosen[1] = bn; chosen[2] = ch.parts; }
  int tiles = 0, blocks = 0;
  float *part0 = scratch;
  for (int i = 0; i < g.n; ++i) {
    TnProduct &p = g.p[i];
    p.tiles_m = (p.M + bm - 1) / bm;
    p.tiles_n = (p.N + bn - 1) / bn;
    p.first = tiles;
    tiles += p.tiles_m * p.tiles_n;
    o.first[i] = blocks;
    blocks += (int)(((int64_t)p.M * p.N + 1023) / 1024);
    if (ch.parts > 1) {
      p.out = part0;
      p.vec_ok = p.N % 4 == 0 && aligned16(part0);
      part0 += (int64_t)ch.parts * p.M * p.N;
    }
  }
  TnGroup run = g;
  if (ch.parts > 1)
    for (int i = 0; i < g.n; ++i) run.p[i].alpha = 1.f;
  Ep ep{1.f, nullptr, nullptr, nullptr, 1, 0, nullptr, 0, 0};
  if (!bf16) {
    F32Product fp[kGroupProducts];
    for (int i = 0; i < g.n; ++i) {
      const TnProduct &p = run.p[i];
      fp[i] = {reinterpret_cast<const float *>(p.a), reinterpret_cast<const float *>(p.b), p.out, p.lda, p.ldb, p.M, p.N, p.first, p.tiles_m, p.tiles_n, p.alpha};
    }
    twist_launch_gemm_f32_group(stream, bm, g.n, fp, tiles, K, ch.parts, ch.kchunk);
  } else if (ch.kind < 2) {
    const dim3 grid(std::min(tiles * ch.parts, 256)), block(512);
    if (ch.kind == 0) hipLaunchKernelGGL((pp::gemm_pp_kernel<0, true, 256, TnGroup>), grid, block, 0, stream, 0, 0, K, nullptr, 0, nullptr, 0, ep, tiles, 1, ch.parts, ch.kchunk, run);
    else hipLaunchKernelGGL((pp::gemm_pp_kernel<0, true, 128, TnGroup>), grid, block, 0, stream, 0, 0, K, nullptr, 0, nullptr, 0, ep, tiles, 1, ch.parts, ch.kchunk, run);
  } else if (ch.kind < kOneGroup) {
    twist_launch_gemm_dl_group(stream, ch.kind == 2 ? 64 : 32, &run, tiles, K, &ep, ch.parts, ch.kchunk);
  } else {
    twist_launch_gemm_kp_group(stream, bm, bn, &run, tiles, K, &ep, ch.parts, ch.kchunk);
  }
  TW_HIP(ctx, hipGetLastError());
  if (ch.parts > 1) {
    hipLaunchKernelGGL(group_reduce_kernel, dim3(blocks), dim3(256), 0, stream, g, o, ch.parts);
    TW_HIP(ctx, hipGetLastError());
  }
  return TWIST_OK;
}

void twist_gemm_estimate(GemmLayout lay, int n, const int *Ms, const int *Ns, int K, bool f32_out, size_t split_floats, GemmEstimate &sum) {
  const Choice ch = choose_any(lay, n, Ms, Ns, K, f32_out, split_floats > 0, split_floats);
  sum.us += ch.us;
  sum.idle += ch.idle;
}

extern "C" twist_status twist_gemm_raw(twist_ctx *ctx, int32_t layout, int32_t M, int32_t N, int32_t K, const void *A, int64_t lda, const void *B,
                                       int64_t ldb, void *C, int64_t ldc, int32_t out_f32, float alpha) {
  return twist_gemm_raw_cut(ctx, layout, M, N, K, A, lda, B, ldb, C, ldc, out_f32, alpha, nullptr, 0);
}

extern "C" twist_status twist_gemm_raw_cut(twist_ctx *ctx, int32_t layout, int32_t M, int32_t N, int32_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
                                           void *C, int64_t ldc, int32_t out_f32, float alpha, float *scratch, size_t scratch_floats) {
  if (!ctx || !A || !B || !C) TW_FAIL(ctx, TWIST_EINVAL, "twist_gemm_raw: null argument");
  if (layout < 0 || layout > 2 || M < 0 || N < 0 || K < 0) TW_FAIL(ctx, TWIST_EINVAL, "twist_gemm_raw: bad layout or size");
  const int64_t need_a = layout == GEMM_TN ? M : K, need_b = layout == GEMM_NT ? K : N;
  if (lda < need_a || ldb < need_b || ldc < N) TW_FAIL(ctx, TWIST_ESHAPE, "twist_gemm_raw: a row stride is smaller than the row it strides");
  if (!aligned16(scratch)) TW_FAIL(ctx, TWIST_ESHAPE, "twist_gemm_raw_cut: the scratch must be 16-byte aligned");
  GemmEpilogue e;
  e.alpha = alpha;
  e.out = C;
  e.out_f32 = out_f32;
  e.splitk_ws = scratch;
  e.splitk_floats = scratch_floats;
  return twist_gemm(ctx, ctx->d.dtype == TWIST_BF16, (GemmLayout)layout, M, N, K, A, lda, B, ldb, ldc, e);
}

extern "C" twist_status twist_gemm_act_raw(twist_ctx *ctx, int32_t layout, int32_t M, int32_t N, int32_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
                                           void *C, int64_t ldc, const void *bias, int32_t act, void *act_out, int32_t act_only) {
  if (!ctx || !A || !B || !C || !act_out) TW_FAIL(ctx, TWIST_EINVAL, "twist_gemm_act_raw: null argument");
  if (layout < 0 || layout > 2 || M < 0 || N < 0 || K < 0) TW_FAIL(ctx, TWIST_EINVAL, "twist_gemm_act_raw: bad layout or size");
  const int64_t need_a = layout == GEMM_TN ? M : K, need_b = layout == GEMM_NT ? K : N;
  if (lda < need_a || ldb < need_b || ldc < N) TW_FAIL(ctx, TWIST_ESHAPE, "twist_gemm_act_raw: a row stride is smaller than the row it strides");
  GemmEpilogue e;
  e.bias = bias;
  e.out = C;
  e.act_out = act_out;
  e.act = act;
  e.act_only = act_only != 0;
  return twist_gemm(ctx, ctx->d.dtype == TWIST_BF16, (GemmLayout)layout, M, N, K, A, lda, B, ldb, ldc, e);
}

extern "C" twist_status twist_weight_grads_raw(twist_ctx *ctx, int32_t n, const twist_weight_grad *products, int32_t K, float *scratch, size_t scratch_floats,
                                               int32_t chosen[3]) {
  if (!ctx || !products) TW_FAIL(ctx, TWIST_EINVAL, "twist_weight_grads_raw: null argument");
  if (n < 1 || n > kGroupProducts || K < 0) TW_FAIL(ctx, TWIST_EINVAL, "twist_weight_grads_raw: bad number of products or rows");
  for (int i = 0; i < n; ++i) {
    const twist_weight_grad &p = products[i];
    if (p.M < 0 || p.N < 0 || (p.M > 0 && p.N > 0 && (!p.a || !p.b || !p.out))) TW_FAIL(ctx, TWIST_EINVAL, "twist_weight_grads_raw: bad product %d", i);
    if (p.lda < p.M || p.ldb < p.N) TW_FAIL(ctx, TWIST_ESHAPE, "twist_weight_grads_raw: a row stride is smaller than the row it strides");
  }
  if (!aligned16(scratch)) TW_FAIL(ctx, TWIST_ESHAPE, "twist_weight_grads_raw: the scratch must be 16-byte aligned");
  if (chosen) chosen[0] = chosen[1] = chosen[2] = 0;
  return twist_weight_grads(ctx, ctx->d.dtype == TWIST_BF16, n, products, K, scratch, scratch_floats, nullptr, chosen);
}

extern "C" twist_status twist_gemm_kernel(twist_ctx *ctx, int32_t layout, int32_t M, int32_t N, int32_t K, int32_t out_f32, size_t scratch_floats, int32_t chosen[3]) {
  if (!ctx || !chosen) TW_FAIL(ctx, TWIST_EINVAL, "twist_gemm_kernel: null argument");
  if (layout < 0 || layout > 2 || M < 1 || N < 1 || K < 1) TW_FAIL(ctx, TWIST_EINVAL, "twist_gemm_kernel: bad layout or size");
  if (ctx->d.dtype == TWIST_BF16) {
    const Cut ch = cut_of(ctx, true, (GemmLayout)layout, M, N, K, out_f32, scratch_floats > 0, scratch_floats);
    chosen[0] = kKinds[ch.kind].bm; chosen[1] = kKinds[ch.kind].bn; chosen[2] = ch.parts;
  } else if (short_f32(ctx, (GemmLayout)layout, M, N, K)) {
    chosen[0] = chosen[1] = 0; chosen[2] = 1;
  } else {
    int kchunk;
    twist_gemm_f32_choice(ctx, (GemmLayout)layout, M, N, K, dense_rows_of_16((GemmLayout)layout, M, N, K), scratch_floats > 0, scratch_floats, chosen[0], chosen[2], kchunk);
    chosen[1] = chosen[0];
  }
  return TWIST_OK;
}
extern "C" twist_status twist_gemm_tile(twist_ctx *ctx, int32_t layout, int32_t M, int32_t N, int32_t K, int32_t out_f32, size_t scratch_floats, int32_t chosen[3]) {
  return twist_gemm_kernel(ctx, layout, M, N, K, out_f32, scratch_floats, chosen);
}

extern "C" twist_status twist_set_overlap(twist_ctx *ctx, int32_t enable) {
  if (!ctx) TW_FAIL(nullptr, TWIST_EINVAL, "twist_set_overlap: null ctx");
  ctx->overlap = enable != 0;
  return TWIST_OK;
}

extern "C" twist_status twist_set_kernel_choice(twist_ctx *ctx, int32_t gemm_tile, int32_t plain_only, int32_t staged_attention) {
  if (!ctx) TW_FAIL(nullptr, TWIST_EINVAL, "twist_set_kernel_choice: null ctx");
  if (gemm_tile != 0 && gemm_tile != 128 && gemm_tile != 256) TW_FAIL(ctx, TWIST_EINVAL, "twist_set_kernel_choice: gemm_tile must be 0, 128 or 256");
  ctx->gemm_tile = gemm_tile;
  ctx->plain_only = plain_only != 0;
  ctx->staged_attention = staged_attention != 0;
  return TWIST_OK;
}

extern "C" twist_status twist_profile_mfma_ceiling(twist_ctx *ctx, int32_t waves_per_simd, int32_t iters, int32_t random_operands, float *sink,
                                                   size_t sink_floats, double *tflops) {
  if (!ctx || !sink || !tflops) TW_FAIL(ctx, TWIST_EINVAL, "twist_profile_mfma_ceiling: null argument");
  if (waves_per_simd < 1 || waves_per_simd > 8 || iters < 1) TW_FAIL(ctx, TWIST_EINVAL, "twist_profile_mfma_ceiling: waves_per_simd in [1, 8], iters >= 1");
  hipDeviceProp_t prop;
  int dev = 0;
  TW_HIP(ctx, hipGetDevice(&dev));
  TW_HIP(ctx, hipGetDeviceProperties(&prop, dev));
  const int blocks = prop.multiProcessorCount * waves_per_simd;  // a workgroup is 4 waves, one per SIMD of a compute unit
  if (sink_floats < (size_t)blocks * 256) TW_FAIL(ctx, TWIST_ESHAPE, "twist_profile_mfma_ceiling: sink needs %zu floats", (size_t)blocks * 256);
  hipEvent_t e0, e1;
  TW_HIP(ctx, hipEventCreate(&e0));
  TW_HIP(ctx, hipEventCreate(&e1));
  hipLaunchKernelGGL(mfma_only_kernel, dim3(blocks), dim3(256), 0, ctx->stream, iters / 8 + 1, sink, random_operands);  // warm-up
  (void)hipEventRecord(e0, ctx->stream);
  hipLaunchKernelGGL(mfma_only_kernel, dim3(blocks), dim3(256), 0, ctx->stream, iters, sink, random_operands);
  (void)hipEventRecord(e1, ctx->stream);
  hipError_t err = hipEventSynchronize(e1);
  float ms = 0.f;
  if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  TW_HIP(ctx, err);
  const double trips = (double)((iters + 3) / 4);  // the kernel runs four iterations per trip
  *tflops = (double)blocks * 4.0 * trips * 16.0 * (2.0 * 32 * 32 * 16) / ((double)ms * 1e-3) / 1e12;
  return TWIST_OK;
}

extern "C" twist_status twist_profile_gemm(twist_ctx *ctx, int32_t enable) {
  if (!ctx) TW_FAIL(nullptr, TWIST_EINVAL, "twist_profile_gemm: null ctx");
  TW_HIP(ctx, hipStreamSynchronize(ctx->stream));
  for (hipEvent_t e : ctx->prof_events) (void)hipEventDestroy(e);
  ctx->prof_events.clear();
  ctx->prof_flops = 0.0;
  ctx->prof_gemm = enable != 0;
  return TWIST_OK;
}

extern "C" twist_status twist_profile_gemm_read(twist_ctx *ctx, int64_t *launches, double *ms, double *flops) {
  if (!ctx || !launches || !ms || !flops) TW_FAIL(ctx, TWIST_EINVAL, "twist_profile_gemm_read: null argument");
  TW_HIP(ctx, hipStreamSynchronize(ctx->stream));
  double total = 0.0;
  for (size_t i = 0; i + 1 < ctx->prof_events.size(); i += 2) {
    float t = 0.f;
    TW_HIP(ctx, hipEventElapsedTime(&t, ctx->prof_events[i], ctx->prof_events[i + 1]));
    total += t;
  }
  *launches = (int64_t)(ctx->prof_events.size() / 2);
  *ms = total;
  *flops = ctx->prof_flops;
  for (hipEvent_t e : ctx->prof_events) (void)hipEventDestroy(e);
  ctx->prof_events.clear();
  ctx->prof_flops = 0.0;
  return TWIST_OK;
}
