// Dense projections of fp32 models on the matrix cores.
//
// Tiles of 128 and 64: gemm_f32_kernel and gemm_f32_wave_kernel, on the bf16 instruction (v_mfma_f32_32x32x16_bf16, sixteen times the rate of the fp32 one).  An fp32
// value is the sum of three bf16 values (8 bits each, rounded to nearest, the last one exactly what is left), a product of two bf16 values is exact in
// fp32, and of the nine products of two such sums the six largest are formed.  What is left out of a product is 2^-28 of it on average over
// operands of random bits and at most about 2^-24 (0.99 of that for the square of 1 + 2^-8 - 2^-17), one rounding of fp32.  The sums run in fp32 as
// before, in fewer steps (one per 16 products), the small products in a sum of their own.  Error against 64 bits on normal operands, the fp32
// instruction in brackets: K = 17 0.4e-7 (0.8e-7), 33 0.4e-7 (1.0e-7), 100 0.5e-7 (1.8e-7), 384 0.8e-7 (1.8e-7), 768 1.1e-7 (2.5e-7 to 5.0e-7),
// 4096 2.7e-7 (11.5e-7), 50257 in 16 parts 2.5e-7 (10e-7); one sum for all six products: K = 768 3.0e-7.
// The third term of a value below 2^-110 would need bits below the smallest bf16 (2^-133; the instruction takes subnormal operands), so the terms
// are those of 2^16 times the value, which holds down to the smallest fp32 (2^-149), and 2^32 is taken out of the sums: operands of 1e-36 0.7e-7
// (without the factor 270e-7).
// Tiles of 32, for few rows: gemm_f32_small_kernel, on the fp32 instruction (v_mfma_f32_32x32x2_f32): there every value would be split into
// its terms for 32 products only.
//
// gemm_f32_wave_kernel, tiles of 64 whose operands allow 16-byte loads, contractions from 320 on and some shorter ones (launch_tile).  What bounded such tiles in gemm_f32_kernel was neither the matrix
// pipes nor the loads but LDS and what it is fed with: three terms of 2 bytes written and, by waves of 32x32, read twice, a barrier for every
// slice, and two waves a SIMD in step (1.2 us per slice of 64 where the instructions take 0.35 and forming the terms 0.47).  Here every wave forms
// the whole tile over steps of 16 k of its own, so that
//  - no two waves need the same element: it crosses LDS once, as fp32, and its terms are formed in the registers that multiply it;
//  - there is no barrier before the waves' sums are added at the end: while one wave of a SIMD forms terms the other multiplies;
//  - a wave's next two steps are in flight, loaded straight to LDS in whole pieces of rows (a first form that loaded the fragments into
//    registers spent its time on the addresses of 32 rows per load: 1024 x 768 x 1536 48 us).
// Its chains are an eighth (a quarter) of the contraction long, and the error is smaller: K = 96 0.47e-7 (gemm_f32_kernel 0.53e-7), 768 0.8e-7 (1.1e-7),
// 4096 1.9e-7 (2.7e-7), 50257 whole 5.0e-7 (10e-7).  us, before / now: 1024 x 768 x 1536 32.1 / 23.6, its NN form 35.3 / 23.8, 1152 x 768 x 1024 (TN) 25.2 / 18.8,
// 1024 x 1536 x 768 31.6 / 25.5, 1536 x 768 x 1024 (TN) 37.7 / 27.5, 8192 x 768 x 768 89 / 78, 3072 x 768 x 8192 (TN) 330 / 262, 1024 x 768 x 50257 (NN, cut)
// 580 / 490.  What bounds it: small products the fixed 6 us (launch 2, first loads 2, sums and stores 2), large ones the power limit: 4096^3 797 us, in
// tiles of 128 824 to 830 on the same card.
//
// gemm_f32_kernel and gemm_f32_small_kernel: four or eight waves, the contraction walked in slices of BK that are double-buffered in LDS, one
// barrier per slice.  The waves divide the tile, and (WK) the slice: their results are added in wave order at the end.
// gemm_f32_kernel: three slices are in flight to registers; their terms are formed on the way to LDS, in the orientation of the memory:
//   k contiguous ("KM"): [rows][BK + 8], plain 16-byte fragment reads;      rows contiguous: [BK][rows + 16], transposing reads.
// gemm_f32_small_kernel: one slice in flight;
//   k contiguous: LDS [rows][BK + 4], a lane reads 4 consecutive k at once, good for four MFMAs;      rows contiguous: [BK][rows + 8].
//   MFMA number 4 u + j of a slice contracts k = 8 u + j (lanes 0-31) and 8 u + 4 + j (lanes 32-63): the order of k inside a slice
//   is free as long as both operands agree.  Both paddings make the reads conflict-free.
// Measured, us (before: the fp32 instruction in all tiles), tiles of 128, on another card than the figures above: 4096^3 805 (1107), 4096 x 2048 x 2048 222
// (286), 1024 x 50257 x 768 595 (741): the rate of the bf16 instruction at the power limit (six of them per product: 1.04 PFLOP/s in 4096^3).  All three run on
// tiles of 64 now (1024 x 50257 x 768 560).
// Strides and bases that do not allow 16-byte loads go through the scalar loader (VEC = 0), in tiles of 64 too.
#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"

namespace {

constexpr float kUp = 65536.f, kDown = 1.f / (kUp * kUp);  // factor of the terms, and what takes it out of a sum of their products
// four floats as three vectors of bf16 that add up to kUp times them exactly (an infinity, a NaN or what overflows gives a NaN)
__device__ __forceinline__ void split(f32x4 v, u32x2 (&t)[3]) {
  v *= kUp;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    t[k] = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    if (k == 2) break;
    v[0] -= __uint_as_float(t[k].x << 16);
    v[1] -= __uint_as_float(t[k].x & 0xffff0000u);
    v[2] -= __uint_as_float(t[k].y << 16);
    v[3] -= __uint_as_float(t[k].y & 0xffff0000u);
  }
}

// for the fp32 instruction: four consecutive k of one row, from a slice in LDS stored by rows (KM) or by k
template <int KM, int LD>
__device__ __forceinline__ f32x4 four_k(const float *lds, int row, int k) {
  if (KM) return *reinterpret_cast<const f32x4 *>(lds + row * LD + k);
  const float *p = lds + k * LD + row;
  return f32x4{p[0], p[LD], p[2 * LD], p[3 * LD]};
}

constexpr int kAhead = 3;  // slices in flight between memory and registers

// One operand's slice: fp32 from memory to registers, its three terms to LDS, fragments of 32 rows x 16 k back
template <int ROWS, int KM, int VEC, int BK, int NT>
struct Loader {
  static constexpr int LD = KM ? BK + 8 : ROWS + 16;            // elements of a stored row
  static constexpr int PLANE = KM ? ROWS * LD : BK * LD;        // elements of one term
  static constexpr int ELEMS = 3 * PLANE;
  static constexpr int CHUNKS = ROWS * BK / 4 / NT;             // groups of 4 floats per thread (NT threads)
  static constexpr int CPR = KM ? BK / 4 : ROWS / 4;            // groups per stored row
  f32x4 reg[kAhead][CHUNKS];  // slices on their way
  const float *base;
  uint32_t off[CHUNKS];    // byte offset of this thread's groups from the slice's first element (32 bits: the caller checks the range)
  int64_t step;            // floats from one slice to the next
  int rows_left;
  // base = first row of the panel (KM) or first column (otherwise) at the first k
  __device__ __forceinline__ void init(const float *base_, int64_t ld, int rows_left_) {
    base = base_;
    step = KM ? BK : BK * ld;
    rows_left = rows_left_;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = threadIdx.x + NT * i, major = c / CPR, minor = (c % CPR) * 4;
      // rows beyond the last give results that are not stored: they are read from the last (KM) or from the last group that holds a row
      const int r = KM ? min(major, rows_left - 1) : min(minor, (rows_left - 1) / 4 * 4);
      off[i] = (uint32_t)((KM ? r * ld + minor : major * ld + r) * 4);
    }
  }
  // the next slice's groups into register set `set`; k_left = k from the slice's first to the end of the contraction
  __device__ __forceinline__ void load(int set, int k_left) {
    if (VEC && k_left >= BK && (KM || rows_left >= ROWS)) {
#pragma unroll
      for (int i = 0; i < CHUNKS; ++i) reg[set][i] = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const char *>(base) + off[i]);
    } else {
#pragma unroll
      for (int i = 0; i < CHUNKS; ++i) {
        const int c = threadIdx.x + NT * i, k = KM ? c % CPR * 4 : c / CPR, r = KM ? 0 : min(c % CPR * 4, (rows_left - 1) / 4 * 4);
        const float *p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + off[i]);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        // what lies beyond the last k is zero; (an aligned group that straddles an edge holds at least one element of the operand, so reading it is safe)
        if (VEC && k < k_left) v = *reinterpret_cast<const f32x4 *>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = KM ? k + e < k_left : (k < k_left && r + e < rows_left);
          if (VEC) v[e] = in ? v[e] : 0.f;
          else if (in) v[e] = p[e];
        }
        reg[set][i] = v;
      }
    }
    base += step;
  }
  __device__ __forceinline__ void store(int set, uint16_t *lds) const {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = threadIdx.x + NT * i;
      u32x2 t[3];
      split(reg[set][i], t);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2 *>(lds + k * PLANE + (c / CPR) * LD + (c % CPR) * 4) = t[k];
    }
  }
  // register set 0 as it is, for the fp32 instruction
  static constexpr int LD32 = KM ? BK + 4 : ROWS + 8, ELEMS32 = KM ? ROWS * LD32 : BK * LD32;
  __device__ __forceinline__ void store_f32(float *lds) const {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = threadIdx.x + NT * i;
      *reinterpret_cast<f32x4 *>(lds + (c / CPR) * LD32 + (c % CPR) * 4) = reg[0][i];
    }
  }
  // the wave's fragments of the 32 rows from row0 on and the 16 k from k0 on, all three terms
  static __device__ __forceinline__ void frag(const uint16_t *lds, int row0, int k0, bf16x8 (&f)[3]) {
    const int lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5, s = lane & 15, hi = (lane >> 4) & 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (KM) {
        f[k] = *reinterpret_cast<const bf16x8 *>(lds + k * PLANE + (row0 + c) * LD + k0 + 8 * g);
      } else {
        typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
        const uint16_t *q = lds + k * PLANE + (k0 + 8 * g + (s >> 2)) * LD + row0 + 16 * hi + 4 * (s & 3);
        const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q)), y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(q + 4 * LD));
        f[k] = __builtin_bit_cast(bf16x8, s16x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]});
      }
    }
  }
};

template <int ROWS, int KM, int VEC, int BK>
struct SmallLoader {
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
    return four_k<KM, LD>(lds, row0 + (threadIdx.x & 31), 8 * u + 4 * ((threadIdx.x >> 5) & 1));
  }
};

struct Ep32 {
  float alpha;
  const float *bias, *residual;
  float *out;
  int64_t ldc;
};

// Weight gradients that share a launch: with G = F32Group their sizes, operands and outputs replace the kernels' arguments, and tiles_m is the
// number of tiles of all of them.
struct F32Group {
  int n;
  F32Product p[kGroupProducts];
};
template <class G>
__device__ __forceinline__ void take_product(const G &group, int &bid, int &M, int &N, const float *&A, int64_t &lda, const float *&B, int64_t &ldb, Ep32 &ep,
                                             int &tiles_m, int &tiles_n) {
  if constexpr (std::is_same<G, F32Group>::value) {
    int q = 0;
#pragma unroll
    for (int i = 1; i < kGroupProducts; ++i)
      if (i < group.n && bid >= group.p[i].first) q = i;
    const F32Product &p = group.p[q];
    bid -= p.first;
    M = p.M; N = p.N; A = p.a; lda = p.lda; B = p.b; ldb = p.ldb; tiles_m = p.tiles_m; tiles_n = p.tiles_n;
    ep.alpha = p.alpha; ep.out = p.out; ep.ldc = N;
  }
}

// Waves: 2 x 2 over the tile (W2 = 2) or one (W2 = 1), times WK shares of a slice's k; where two waves share a SIMD (8 waves) the first four
// form the next slice's terms before their products, the others after, so that a SIMD's matrix and vector pipes are busy together.
// Grid: x = tiles (dealt so that each of the 8 XCDs walks a contiguous range, in columns of 8 tile rows), y = parts of the
// contraction (kchunk long, a multiple of BK; part p writes its partial product to out + p M ldc).
template <int AKM, int BKM, int BM, int W2, int WK, int BK, int VEC, class G = NoGroup>
__global__ __launch_bounds__(64 * W2 * W2 * WK) void gemm_f32_kernel(int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, Ep32 ep, int tiles_m,
                                                                     int tiles_n, int kchunk, G group) {
  constexpr int BN = BM, NT = 64 * W2 * W2 * WK, TM = BM / W2 / 32, KS = BK / 16 / WK;  // TM: 32x32 tiles of a wave each way; KS: its steps of 16 k per slice
  using LA = Loader<BM, AKM, VEC, BK, NT>;
  using LB = Loader<BN, BKM, VEC, BK, NT>;
  constexpr int STAGE = LA::ELEMS + LB::ELEMS;
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * STAGE];
  const int nb = tiles_m * tiles_n;
  int bid = blockIdx.x;
  if (nb % 8 == 0) bid = (bid % 8) * (nb / 8) + bid / 8;
  take_product(group, bid, M, N, A, lda, B, ldb, ep, tiles_m, tiles_n);
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int m0 = (first_m + (bid % per_group) % gsize) * BM, n0 = ((bid % per_group) / gsize) * BN;
  const int kbeg = blockIdx.y * kchunk, kend = min(K, kbeg + kchunk);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wk = wave / (W2 * W2), wpos = wave % (W2 * W2);
  const int wm = wpos / W2 * (BM / W2), wn = wpos % W2 * (BN / W2), kw = wk * (BK / WK);
  const bool late = W2 * W2 * WK == 8 && wave >= 4;
  const float *pa = AKM ? A + (int64_t)m0 * lda : A + m0, *pb = BKM ? B + (int64_t)n0 * ldb : B + n0;

  f32x16 acc[TM][TM], low[TM][TM];  // the sums of the largest products, and of the others: fewer roundings at the size of the result
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[i][j][r] = 0.f; low[i][j][r] = 0.f; }
  LA la;
  LB lb;
  la.init(AKM ? pa + kbeg : pa + (int64_t)kbeg * lda, lda, M - m0);
  lb.init(BKM ? pb + kbeg : pb + (int64_t)kbeg * ldb, ldb, N - n0);
  la.load(0, kend - kbeg);
  lb.load(0, kend - kbeg);
  la.store(0, lds);
  lb.store(0, lds + LA::ELEMS);
#pragma unroll
  for (int u = 1; u <= kAhead; ++u)
    if (kbeg + u * BK < kend) {
      la.load(u % kAhead, kend - kbeg - u * BK);
      lb.load(u % kAhead, kend - kbeg - u * BK);
    }
  __syncthreads();
  int cur = 0;
  for (int k1 = kbeg; k1 < kend; k1 += kAhead * BK) {
#pragma unroll
  for (int d = 0; d < kAhead; ++d, cur ^= 1) {
    const int k0 = k1 + d * BK;
    if (k0 >= kend) break;
    // slice k0 is in LDS, the next ones in registers or on their way there
    auto next = [&] {
      const int set = (d + 1) % kAhead;
      if (k0 + BK < kend) {
        la.store(set, lds + (cur ^ 1) * STAGE);
        lb.store(set, lds + (cur ^ 1) * STAGE + LA::ELEMS);
      }
      if (k0 + (kAhead + 1) * BK < kend) {
        la.load(set, kend - k0 - (kAhead + 1) * BK);
        lb.load(set, kend - k0 - (kAhead + 1) * BK);
      }
    };
    if (!late) next();
    const uint16_t *st = lds + cur * STAGE;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 af[TM][3], bf[TM][3];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        LA::frag(st, wm + i * 32, kw + 16 * ks, af[i]);
        LB::frag(st + LA::ELEMS, wn + i * 32, kw + 16 * ks, bf[i]);
      }
      // the six largest of the nine products, small ones first
#pragma unroll
      for (int p = 0; p < 6; ++p) {
        constexpr int pa_[6] = {2, 0, 1, 1, 0, 0}, pb_[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j) {
            f32x16 &to = p == 5 ? acc[i][j] : low[i][j];
            to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i][pa_[p]], bf[j][pb_[p]], to, 0, 0, 0);
          }
      }
    }
    if (late) next();
    __syncthreads();
  }
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
  bool finite = true;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] += low[i][j][r];
        finite = finite && __builtin_isfinite(acc[i][j][r]);
        acc[i][j][r] *= kDown;
      }
  if (__syncthreads_or(!finite)) {
    // an infinity or a NaN among the operands (or a value beyond 2^111 or a sum beyond 2^95, where the factor overflows): its terms do not behave
    // like it, so this tile is formed again on the fp32 instruction (1024 x 50257 x 768, us: 667, with one NaN in one row of 1024,
    // i.e. in an eighth of the tiles, 934, with nothing but NaNs 1301; 1024 x 1536 x 768 30, 56, 56)
    float *sa = reinterpret_cast<float *>(lds), *sb = sa + LA::ELEMS32;
    static_assert((LA::ELEMS32 + LB::ELEMS32) * sizeof(float) <= sizeof(lds), "one slice in fp32 fits the stages");
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    la.init(AKM ? pa + kbeg : pa + (int64_t)kbeg * lda, lda, M - m0);
    lb.init(BKM ? pb + kbeg : pb + (int64_t)kbeg * ldb, ldb, N - n0);
    la.load(0, kend - kbeg);
    lb.load(0, kend - kbeg);
#pragma unroll 1
    for (int k0 = kbeg; k0 < kend; k0 += BK) {
      la.store_f32(sa);
      lb.store_f32(sb);
      __syncthreads();
      if (k0 + BK < kend) {
        la.load(0, kend - k0 - BK);
        lb.load(0, kend - k0 - BK);
      }
#pragma unroll
      for (int u = 0; u < BK / WK / 8; ++u) {
        const int k = kw + 8 * u + 4 * (lane >> 5);
        f32x4 af[TM], bf[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          af[i] = four_k<AKM, LA::LD32>(sa, wm + 32 * i + (lane & 31), k);
          bf[i] = four_k<BKM, LB::LD32>(sb, wn + 32 * i + (lane & 31), k);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i][e], bf[j][e], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  }
  // the WK shares are added in order; each of their waves finishes 16 / WK of a 32x32 tile's registers
  float *part = reinterpret_cast<float *>(lds);
  constexpr int TILE_F = W2 * W2 * WK * 1024;
  static_assert(sizeof(lds) >= (TM > 1 ? 2 : 1) * TILE_F * sizeof(float), "the results of one 32x32 tile of every wave fit the stages, and of the next");
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int n = n0 + wn + 32 * j + (lane & 31);
    const float bias = ep.bias && n < N ? ep.bias[n] : 0.f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float *p = part + (j * TM + i & 1) * TILE_F + lane;
#pragma unroll
      for (int r = 0; r < 16; ++r) p[wave * 1024 + r * 64] = acc[i][j][r];
      __syncthreads();
#pragma unroll
      for (int rr = 0; rr < 16 / WK; ++rr) {
        const int r = wk * (16 / WK) + rr;
        float x = 0.f;
#pragma unroll
        for (int w = 0; w < WK; ++w) x += p[(w * W2 * W2 + wpos) * 1024 + r * 64];
        if (n < N) put(m0 + wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), n, x, bias);
      }
    }
  }
}

// One operand's 64 rows x 16 k of a wave's step: brought into the wave's own part of LDS as they lie in memory, and read back as fragments.
//   k contiguous: [64 rows][4 chunks of 16 bytes], position p of row r holds chunk p ^ (r / 4) % 4;      rows contiguous: [16 k][64]
template <int KM>
struct Step {
  static constexpr int BYTES = 4096, NP = BYTES / 1024;  // loads of a step
  const float *base;  // the wave's next step: first row of the panel (KM) or first column (otherwise) at its first k
  int64_t ld, step;   // floats from one step of the wave to its next
  int rows;
  f32x4 v[2][2];      // lane (g = lane / 32, c = lane % 32): rows c and 32 + c, k = 8 g .. 8 g + 7
  __device__ __forceinline__ void init(const float *base_, int64_t ld_, int rows_left, int waves) {
    base = base_;
    ld = ld_;
    rows = min(rows_left, 64);
    step = (KM ? 1 : ld) * 16 * waves;
  }
  // start the loads of the next step into st (wave-uniform); k_left > 0: k from its first to the end of the contraction.  Rows (and k, where
  // rows are contiguous) beyond the last lie beyond the buffer's range and come as zeros.  The range ends with a whole chunk: it is aligned
  // and holds at least one element of the operand.
  __device__ __forceinline__ void issue(char *st, int k_left) {
    const int lane = threadIdx.x & 63, up = ((KM ? k_left : rows) + 3) / 4 * 4;
    const desc_t d = make_desc(base, (uint32_t)((((KM ? rows : min(k_left, 16)) - 1) * ld + up) * 4));
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int major = KM ? 16 * i + (lane >> 2) : 4 * i + (lane >> 4), minor = KM ? ((lane & 3) ^ (lane >> 4 & 3)) * 4 : (lane & 15) * 4;
      dma16(d, st + i * 1024, (uint32_t)((major * ld + minor) * 4));
    }
    base += step;
  }
  __device__ __forceinline__ void read(const char *st, int k_left) {
    const int lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (KM) {
          v[i][h] = *reinterpret_cast<const f32x4 *>(st + (32 * i + c) * 64 + (((2 * g + h) ^ (c >> 2 & 3)) << 4));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][h][e] = *reinterpret_cast<const float *>(st + ((8 * g + 4 * h + e) * 64 + 32 * i + c) * 4);
        }
      }
    // what a load brought in beside the operand's own
    if (KM ? k_left < 16 : rows < 64) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][h][e] = (KM ? 8 * g + 4 * h + e < k_left : 32 * i + c < rows) ? v[i][h][e] : 0.f;
    }
  }
  // the three terms of the 32 rows i
  __device__ __forceinline__ void terms(int i, bf16x8 (&t)[3]) const {
    u32x2 a[3], b[3];
    split(v[i][0], a);
    split(v[i][1], b);
#pragma unroll
    for (int k = 0; k < 3; ++k) t[k] = __builtin_bit_cast(bf16x8, u32x4{a[k].x, a[k].y, b[k].x, b[k].y});
  }
};

// Tiles of 64 x 64: every wave forms the whole tile over steps of 16 k of its own (w, w + NW, ...).  One tile per CU: eight waves; more: four,
// two workgroups to a CU.  Grid as in gemm_f32_kernel.
template <int AKM, int BKM, int NW, class G = NoGroup>
__global__ __launch_bounds__(64 * NW, 2) void gemm_f32_wave_kernel(int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, Ep32 ep, int tiles_m,
                                                                   int tiles_n, int kchunk, G group) {
  __shared__ __attribute__((aligned(1024))) f32x4 part[NW][16][64];  // a wave's two steps on their way, and its sums at the end
  const int nb = tiles_m * tiles_n;
  int bid = blockIdx.x;
  if (nb % 8 == 0) bid = (bid % 8) * (nb / 8) + bid / 8;
  take_product(group, bid, M, N, A, lda, B, ldb, ep, tiles_m, tiles_n);
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int m0 = (first_m + (bid % per_group) % gsize) * 64, n0 = ((bid % per_group) / gsize) * 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kend = min(K, (int)(blockIdx.y + 1) * kchunk), kfirst = blockIdx.y * kchunk + 16 * wave;
  const float *pa = AKM ? A + (int64_t)m0 * lda + kfirst : A + (int64_t)kfirst * lda + m0, *pb = BKM ? B + (int64_t)n0 * ldb + kfirst : B + (int64_t)kfirst * ldb + n0;
  Step<AKM> a;
  Step<BKM> b;
  constexpr int STAGE = a.BYTES + b.BYTES, LPS = a.NP + b.NP;
  static_assert(2 * STAGE == sizeof(part[0]), "two steps in flight");
  char *const own = reinterpret_cast<char *>(part[wave]);
  a.init(pa, lda, M - m0, NW);
  b.init(pb, ldb, N - n0, NW);
  auto issue = [&](int slot, int k) {
    a.issue(own + slot * STAGE, kend - k);
    b.issue(own + slot * STAGE + a.BYTES, kend - k);
  };
  auto read = [&](int slot, int k) {
    a.read(own + slot * STAGE, kend - k);
    b.read(own + slot * STAGE + a.BYTES, kend - k);
  };

  f32x16 acc[2][2], low[2][2];  // the sums of the largest products, and of the others: fewer roundings at the size of the result
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[i][j][r] = 0.f; low[i][j][r] = 0.f; }
  if (kfirst < kend) issue(0, kfirst);
  if (kfirst + 16 * NW < kend) issue(1, kfirst + 16 * NW);
  int slot = 0;
#pragma unroll 1
  for (int k = kfirst; k < kend; k += 16 * NW, slot ^= 1) {
    if (k + 16 * NW < kend) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    read(slot, k);
    bf16x8 ta[2][3], tb[2][3];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a.terms(i, ta[i]);
      b.terms(i, tb[i]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the step is in registers: its place is free
    if (k + 32 * NW < kend) issue(slot, k + 32 * NW);
    __builtin_amdgcn_sched_barrier(0);
    // the six largest of the nine products, small ones first
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      constexpr int pa_[6] = {2, 0, 1, 1, 0, 0}, pb_[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f32x16 &to = p == 5 ? acc[i][j] : low[i][j];
          to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ta[i][pa_[p]], tb[j][pb_[p]], to, 0, 0, 0);
        }
    }
  }
  bool finite = true;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[i][j][r] += low[i][j][r];
        finite = finite && __builtin_isfinite(acc[i][j][r]);
        acc[i][j][r] *= kDown;
      }
  if (__syncthreads_or(!finite)) {
    // as in gemm_f32_kernel: the tile is formed again on the fp32 instruction, whose product number 4 h + e of a step contracts k = 4 h + e
    // (lanes 0-31) and 8 + 4 h + e (lanes 32-63)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    a.base = pa;
    b.base = pb;
#pragma unroll 1
    for (int k = kfirst; k < kend; k += 16 * NW) {
      issue(0, k);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      read(0, k);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[i][h][e], b.v[j][h][e], acc[i][j], 0, 0, 0);
    }
  }
  // the waves' sums are added, of eight waves the first pairs in 32 bits, the rest in 64: contractions of 48 to 200 are a step or two per wave, and
  // their error is that of these additions (K = 96 5.9e-8 in 32 bits and wave order, 5.2e-8 in gemm_f32_kernel).  Each wave finishes 16 / NW of the groups of
  // four registers.  Registers 4 q .. 4 q + 3 of tile (i, j): rows 32 i + 8 q + 4 g .. + 3, column 32 j + c
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[wave][(2 * i + j) * 4 + q][lane] = f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
  __syncthreads();
  float *out = ep.out + (int64_t)blockIdx.y * M * ep.ldc;
#pragma unroll
  for (int t = 0; t < 16 / NW; ++t) {
    const int at = wave * (16 / NW) + t, m = m0 + 32 * (at >> 3) + 8 * (at & 3) + 4 * (lane >> 5), n = n0 + 32 * ((at >> 2) & 1) + (lane & 31);
    f32x4 y[4], x;
#pragma unroll
    for (int w = 0; w < 4; ++w) y[w] = NW == 8 ? part[w][at][lane] + part[(w + 4) % NW][at][lane] : part[w][at][lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = (float)(((double)y[0][e] + y[1][e]) + ((double)y[2][e] + y[3][e]));
    if (n >= N) continue;
    const float bias = ep.bias ? ep.bias[n] : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (m + e >= M) break;
      float v = (x[e] + bias) * ep.alpha;
      const int64_t o = (int64_t)(m + e) * ep.ldc + n;
      if (ep.residual) v += ep.residual[o];
      out[o] = v;
    }
  }
}

// Grid: x = tiles (dealt so that each of the 8 XCDs walks a contiguous range, in columns of 8 tile rows), y = parts of the
// contraction (kchunk long, a multiple of BK; part p writes its partial product to out + p M ldc).
template <int AKM, int BKM, int VEC, class G = NoGroup>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, Ep32 ep, int tiles_m,
                                                       int tiles_n, int kchunk, G group) {
  constexpr int BM = 32, BN = 32, BK = 64, US = BK / 8 / 4;  // US: groups of 4 MFMAs per slice and wave
  using LA = SmallLoader<BM, AKM, VEC, BK>;
  using LB = SmallLoader<BN, BKM, VEC, BK>;
  __shared__ __attribute__((aligned(16))) float As[2][LA::ELEMS];
  __shared__ __attribute__((aligned(16))) float Bs[2][LB::ELEMS];
  const int nb = tiles_m * tiles_n;
  int bid = blockIdx.x;
  if (nb % 8 == 0) bid = (bid % 8) * (nb / 8) + bid / 8;
  take_product(group, bid, M, N, A, lda, B, ldb, ep, tiles_m, tiles_n);
  constexpr int GROUP = 8;
  const int per_group = GROUP * tiles_n;
  const int grp = bid / per_group, first_m = grp * GROUP;
  const int gsize = min(GROUP, tiles_m - first_m);
  const int m0 = (first_m + (bid % per_group) % gsize) * BM, n0 = ((bid % per_group) / gsize) * BN;
  const int kbeg = blockIdx.y * kchunk, kend = min(K, kbeg + kchunk);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int u0 = wave * US;
  const float *pa = AKM ? A + (int64_t)m0 * lda : A + m0, *pb = BKM ? B + (int64_t)n0 * ldb : B + n0;

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
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
    f32x4 af[2], bf[2];
    af[0] = LA::frag(As[cur], 0, u0);
    bf[0] = LB::frag(Bs[cur], 0, u0);
#pragma unroll
    for (int u = 0; u < US; ++u) {
      if (u + 1 < US) {
        af[(u + 1) & 1] = LA::frag(As[cur], 0, u0 + u + 1);
        bf[(u + 1) & 1] = LB::frag(Bs[cur], 0, u0 + u + 1);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[u & 1][e], bf[u & 1][e], acc, 0, 0, 0);
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
  // every wave finishes a quarter of the rows: registers 4 w .. 4 w + 3 of all four waves
  float *part = &As[0][0];
  static_assert(sizeof(As) >= 4 * 1024 * sizeof(float), "four 32x32 results fit the A stages");
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave * 1024 + r * 64 + lane] = acc[r];
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

template <int AKM, int BKM, int BM, int W2, int WK, int BK, int VEC>
void launch(hipStream_t st, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, const Ep32 &ep, int parts, int kchunk) {
  const int tm = (M + BM - 1) / BM, tn = (N + BM - 1) / BM;
  hipLaunchKernelGGL((gemm_f32_kernel<AKM, BKM, BM, W2, WK, BK, VEC>), dim3(tm * tn, parts), dim3(64 * W2 * W2 * WK), 0, st, M, N, K, A, lda, B, ldb, ep, tm, tn, kchunk, NoGroup());
}

constexpr int kWaveK = 320;  // shortest contraction for which tiles of 64 are gemm_f32_wave_kernel's
template <int AKM, int BKM, int VEC>
void launch_tile(hipStream_t st, int tile, bool waves, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb, const Ep32 &ep, int parts,
                 int kchunk) {
  if (tile == 128) return launch<AKM, BKM, 128, 2, 2, 32, VEC>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
  if (tile == 64) {
    const int tm = (M + 63) / 64, tn = (N + 63) / 64;
    const bool one = (int64_t)tm * tn * parts <= 256;
    if constexpr (VEC) {
      // shorter contractions are a few steps to a wave, and the addition of the waves' sums and the fixed time weigh more than what the steps save (us,
      // gemm_f32_kernel / waves: 1024 x 768 x 64 5.8 / 6.7, 3000 x 3072 x 64 28.1 / 30.8, 4096 x 512 x 128 9.5 / 10.3, 192 11.7 / 12.0, 256 13.6 / 14.1; 1024 x 768
      // x 320 10.1 / 9.9, x 384 11.6 / 11.3), but where the last slice of 64 would be half empty (1024 x 768 x 96 7.2 / 7.1, 160, NN, 8.5 / 8.0), or tiles
      // of 128 are what they replace (`waves`)
      if (waves || K >= kWaveK || (one && K > 64 && (K + 31) / 32 % 2 == 1)) {
        if (one) hipLaunchKernelGGL((gemm_f32_wave_kernel<AKM, BKM, 8>), dim3(tm * tn, parts), dim3(512), 0, st, M, N, K, A, lda, B, ldb, ep, tm, tn, kchunk, NoGroup());
        else hipLaunchKernelGGL((gemm_f32_wave_kernel<AKM, BKM, 4>), dim3(tm * tn, parts), dim3(256), 0, st, M, N, K, A, lda, B, ldb, ep, tm, tn, kchunk, NoGroup());
        return;
      }
    }
    // slices of 64; more than one tile per CU: of 32, two workgroups to a CU
    if (one) launch<AKM, BKM, 64, 2, 2, 64, VEC>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
    else launch<AKM, BKM, 64, 2, 2, 32, VEC>(st, M, N, K, A, lda, B, ldb, ep, parts, kchunk);
    return;
  }
  const int tm = (M + 31) / 32, tn = (N + 31) / 32;
  hipLaunchKernelGGL((gemm_f32_small_kernel<AKM, BKM, VEC>), dim3(tm * tn, parts), dim3(256), 0, st, M, N, K, A, lda, B, ldb, ep, tm, tn, kchunk, NoGroup());
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Of the k of a part those that one accumulator of a wave sums up; the error of a product grows with the root of that number.  In tiles of 32, on the fp32
// instruction, it is a quarter of k; their error is 1.8 to 2.2 times that of gemm_f32_kernel, as if it were 2.4 k.
double chain_of(int tile, bool vec, int64_t items, double k) { return tile == 32 ? 2.4 * k : tile == 64 && vec ? k / (items <= 256 ? 8 : 4) : k / 2; }

// Tile and number of parts of the contraction, by estimated time of the kernels above (us); n = items (tiles, times parts) on the busiest of
// 256 CUs.  Operands that allow 16-byte loads, K >= 320 or several products:
//   128: 3 + n (8.4 + 1.55 per slice of 32)
//   64: one a CU 6.3 + (0.55 to 0.77, the whole chip at work) per 64 of the contraction, two 7.4 + (1.2 to 1.55), from then on 4.5 + 2.05 n + 0.745 n,
//   and 0.25 for an odd n, per 64
//   32: 3.4 + 1.4 (n - 4, if more) + (0.2 + 0.355 n) per slice of 64
//   sum of a cut one 4 + its bytes at 4.5 TB/s.
// Fitted to 180 products of 48 to 8000 tiles of 64, K = 64 to 4096 (measured; 128 / 64 / 32): 1024 x 768 x 768 43.4 / 15.4 / -, 1024 x 1024 x 4096 186 / 61 / -,
// 1024 x 1152 x 768 43.6 / 22.6 / 30.4, 2048 x 1024 x 1536 80 / 45 / -, 1536 x 1408 x 768 44.5 / 39.4 / -, 2048 x 2048 x 768 48.5 / 49.6 / -,
// 4096 x 1536 x 768 90 / 70 / -, 4096^3 824 / 797 / -, 512 x 384 x 768 40 / 14 / 10.4; 1500 x 1500 x 2000 (TN) 117 / 93 / -, in two
// parts 133 / 88 / 137, in four 113 / 92 / -; 1024 x 768 x 8000 - / 83 / -, in four parts 111 / 93 / -; 3072 x 768 x 8192 (TN) 396 / 332 / 417, in four 332 / 260 / -.
// Others (64 in gemm_f32_kernel): 128 3 + n (6 + 1.47 per slice of 32); 64 one a CU 4.3 + 1.2 per slice of 64, more in pairs, 2 (1.9 + 0.48 per slice of 32),
// a single one left over in the second round 1.9 + 0.85 per slice, and from then on the rounds run into each other; 32 as above.  Rows contiguous in
// both operands (TN): an eighth more for tiles of 128, a sixth for single ones of 64.
// Several products over the same K that share a launch: their tiles and outputs together.
//
// `longest`: how coarse the sums may be (chain_of).  Operands that allow 16-byte loads are summed no more coarsely than the same product without them: by
// time alone 276 x 500 x 1272 (NN) takes tiles of 32 for 0.5 us less and leaves 1.7e-7 where 64 in four parts leaves 0.8e-7; 740 x 848 x 8704 (NN) 64 whole
// for 128 in 16 parts, 2.0e-7 for 1.25e-7.
struct Choice { int tile, parts; };
Choice choose(GemmLayout lay, int count, const int *Ms, const int *Ns, int K, bool vec, bool may_split, size_t split_floats, double longest = 1e30) {
  Choice best{0, 1};
  double best_us = 1e30, outputs = 0.0;
  for (int i = 0; i < count; ++i) outputs += (double)Ms[i] * Ns[i];
  for (int tile = 128; tile >= 32; tile /= 2) {
    int64_t tiles = 0;
    for (int i = 0; i < count; ++i) tiles += (int64_t)((Ms[i] + tile - 1) / tile) * ((Ns[i] + tile - 1) / tile);
    for (int parts = 1; parts <= 16; parts *= 2) {
      if (parts > 1 && (!may_split || K / parts < 256 || parts * outputs > (double)split_floats)) break;
      const int64_t items = tiles * parts;
      if (chain_of(tile, vec, items, (double)K / parts) > longest) continue;
      const double n = (double)((items + 255) / 256), k = (double)K / parts;
      double us;
      if (tile == 128 && vec) {
        us = 3.0 + n * (8.4 + 1.55 * k / 32);
      } else if (tile == 128) {
        us = 3.0 + n * (6.0 + (lay == GEMM_TN ? 1.65 : 1.47) * k / 32);
      } else if (tile == 32) {
        us = (vec ? 3.4 : 4.0) + 1.4 * std::max(n - 4.0, 0.0) + (0.2 + (vec ? 0.355 : 0.36) * n) * k / 64;
      } else if (vec) {
        us = n == 1 ? 6.3 + (0.55 + 0.22 * items / 256) * k / 64 : n == 2 ? 7.4 + (0.9 + 0.65 * items / 512) * k / 64
                    : 4.5 + 2.05 * n + (0.745 * n + ((int64_t)n % 2 ? 0.25 : 0.0)) * k / 64;
      } else if (n == 1) {
        us = 4.3 + (lay == GEMM_TN ? 1.38 : 1.2) * k / 64;
      } else {
        const double pair = 2 * (1.9 + 0.48 * k / 32), rounds = items / 512.0;
        us = 3.0 + (rounds <= 1 ? pair : rounds <= 1.5 ? pair + 1.9 + 0.85 * k / 32 : rounds <= 2 ? 2 * pair : pair * (rounds + 0.25));
      }
      if (parts > 1) us += vec ? 4.0 + (parts + 1.0) * outputs * 4.0 / 4.5e6 : 3.5 + (parts + 1.0) * outputs * 8.0 / 6e6;
      if (us < best_us) { best_us = us; best = {tile, parts}; }
    }
  }
  return best;
}

}  // namespace

// Contractions below kWaveK whose place is on tiles of 128: whether tiles of 64 by waves that form the whole tile take less, by estimates of both for
// operands that allow 16-byte loads (whole slices; the last round of the waves' steps may be short): 128 3 + n (8.2 + 1.32 per slice of 32), where the
// output is beyond 600 MB 3 + n (7.8 + 1.55 per slice).  Fitted to 314 products of 13 to 1650 MB, K = 64 to 316: of the 107 that the waves take one is slower on them,
// by 2 %, the mean is 0.88, and 41 of those they do not take would be 3 to 13 % faster; us, 128 / 64: 8192 x 768 x 256 39.8 / 32.8, 3000 x 3072 x 240 60 / 48.6, 4352 x
// 50257 x 272 1251 / 1109; on the other side 8192 x 2048 x 224 72.5 / 83, 256 78 / 80.6, 1024 x 50257 x 128 176 / 178, 3000 x 32000 x 256 452 / 483.
static bool waves_shorter(int M, int N, int K) {
  const double n128 = (double)(((int64_t)((M + 127) / 128) * ((N + 127) / 128) + 255) / 256);
  const int64_t n64 = ((int64_t)((M + 63) / 64) * ((N + 63) / 64) + 255) / 256;
  const bool beyond = (double)M * N * 4 > 6e8;
  const double by128 = 3.0 + n128 * ((beyond ? 7.8 : 8.2) + (beyond ? 1.55 : 1.32) * ((K + 31) / 32));
  const double by64 = 4.5 + 2.05 * n64 + (0.745 * n64 + (n64 % 2 ? 0.25 : 0.0)) * std::min((double)((K + 63) / 64), K / 64.0 + 0.35);
  return n64 > 2 && by64 < by128;
}

static Choice choice_of(const twist_ctx *ctx, GemmLayout lay, int M, int N, int K, bool vec, bool may_split, size_t split_floats, bool &waves) {
  waves = false;
  if (ctx->gemm_tile) return {ctx->gemm_tile == 128 ? 128 : 64, 1};
  const Choice ch = choose(lay, 1, &M, &N, K, false, may_split, split_floats);
  if (!vec) return ch;
  if (K >= kWaveK) return choose(lay, 1, &M, &N, K, true, may_split, split_floats, chain_of(ch.tile, false, 0, (double)K / ch.parts));
  waves = ch.tile == 128 && waves_shorter(M, N, K);
  return waves ? Choice{64, 1} : ch;
}

static void cut_of(Choice ch, int K, int &tile, int &parts, int &kchunk) {
  const int bk = ch.tile == 128 ? 32 : 64;
  kchunk = ((K + ch.parts - 1) / ch.parts + bk - 1) / bk * bk;
  tile = ch.tile;
  parts = (K + kchunk - 1) / kchunk;
}

void twist_gemm_f32_choice(const twist_ctx *ctx, GemmLayout lay, int M, int N, int K, bool vec, bool may_split, size_t split_floats, int &tile, int &parts, int &kchunk) {
  bool waves;
  cut_of(choice_of(ctx, lay, M, N, K, vec, may_split, split_floats, waves), K, tile, parts, kchunk);
}

twist_status twist_gemm_f32(twist_ctx *ctx, hipStream_t st, GemmLayout lay, int M, int N, int K, const float *A, int64_t lda, const float *B, int64_t ldb,
                            int64_t ldc, const GemmEpilogue &e) {
  Ep32 ep{e.alpha, static_cast<const float *>(e.bias), e.residual, static_cast<float *>(e.out), ldc};
  const bool vec = aligned16(A) && aligned16(B) && lda % 4 == 0 && ldb % 4 == 0;
  int tile, parts, kchunk;
  bool waves;
  cut_of(choice_of(ctx, lay, M, N, K, vec, e.splitk_ws && !e.bias && !e.residual, e.splitk_floats, waves), K, tile, parts, kchunk);
  if (tile != 32 && std::max(lda, ldb) >= 1 << 23) {  // a slice of such rows exceeds the larger tiles' 32-bit offsets
    tile = 32;
    kchunk = (kchunk + 63) / 64 * 64;
    parts = (K + kchunk - 1) / kchunk;
  }
  if (parts > 1) ep = Ep32{1.f, nullptr, nullptr, e.splitk_ws, N};
#define TW_F32(AKM, BKM)                                                                                \
  do {                                                                                                    \
    if (vec) launch_tile<AKM, BKM, 1>(st, tile, waves, M, N, K, A, lda, B, ldb, ep, parts, kchunk);              \
    else launch_tile<AKM, BKM, 0>(st, tile, false, M, N, K, A, lda, B, ldb, ep, parts, kchunk);                  \
  } while (0)
  switch (lay) {
    case GEMM_NT: TW_F32(1, 1); break;
    case GEMM_NN: TW_F32(1, 0); break;
    case GEMM_TN: TW_F32(0, 0); break;
  }
#undef TW_F32
  TW_HIP(ctx, hipGetLastError());
  if (parts > 1) return twist_splitk_reduce(ctx, st, e.splitk_ws, parts, M, N, e.out, ldc, 1, e.alpha);
  return TWIST_OK;
}

// As with a single product, a common launch is no coarser in its sums than every product by itself on unaligned rows: 280 x 1120 and 1120 x 280 over 1636
// rows on tiles of 32 would have an error of 3.7e-7 instead of 1.9e-7.  False where the scratch does not hold that many parts.
bool twist_gemm_f32_group_choice(int n, const int *Ms, const int *Ns, int K, size_t split_floats, int &tile, int &parts, int &kchunk) {
  double longest = 1e30;
  for (int i = 0; i < n; ++i) {
    const Choice c = choose(GEMM_TN, 1, Ms + i, Ns + i, K, false, split_floats > 0, split_floats);
    longest = std::min(longest, chain_of(c.tile, false, 0, (double)K / c.parts));
  }
  const Choice ch = choose(GEMM_TN, n, Ms, Ns, K, true, split_floats > 0, split_floats, longest);
  if (!ch.tile) return false;
  cut_of(ch, K, tile, parts, kchunk);
  return true;
}

void twist_launch_gemm_f32_group(hipStream_t st, int tile, int n, const F32Product *products, int tiles, int K, int parts, int kchunk) {
  F32Group g{};
  g.n = n;
  for (int i = 0; i < n; ++i) g.p[i] = products[i];
  const Ep32 ep{1.f, nullptr, nullptr, nullptr, 0};
#define TW_F32G(BM, BK) hipLaunchKernelGGL((gemm_f32_kernel<0, 0, BM, 2, 2, BK, 1, F32Group>), dim3(tiles, parts), dim3(512), 0, st, 0, 0, K, nullptr, 0, nullptr, 0, ep, tiles, 1, kchunk, g)
#define TW_F32W(NW) hipLaunchKernelGGL((gemm_f32_wave_kernel<0, 0, NW, F32Group>), dim3(tiles, parts), dim3(64 * NW), 0, st, 0, 0, K, nullptr, 0, nullptr, 0, ep, tiles, 1, kchunk, g)
  if (tile == 128) TW_F32G(128, 32);
  else if (tile == 64 && (int64_t)tiles * parts <= 256) TW_F32W(8);
  else if (tile == 64) TW_F32W(4);
  else hipLaunchKernelGGL((gemm_f32_small_kernel<0, 0, 1, F32Group>), dim3(tiles, parts), dim3(256), 0, st, 0, 0, K, nullptr, 0, nullptr, 0, ep, tiles, 1, kchunk, g);
#undef TW_F32W
#undef TW_F32G
}
