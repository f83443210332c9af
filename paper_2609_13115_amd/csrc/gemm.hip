// Projection and rotation GEMMs on the matrix cores (Sec. V-B.3: the
// Rayleigh-Ritz projection H_s = Psi_f^T (H Psi_f), M_s = Psi_f^T Psi_f and the
// subspace rotation Psi = Psi_f Y are dense products).
//
//   gemm_tn : C = A^T B with a long inner dimension K = N_d, split along K
//             (each split's partial tile is written in FP64 and the splits are
//             summed in a fixed order: deterministic, no atomics).
//   gemm_nn : C = A B with A the tall N_d x N_s block and B the N_s x N_s
//             rotation.
// Arithmetic forms (all accumulate in the MFMA accumulator type):
//   FP64  v_mfma_f64_16x16x4f64 (FP32 inputs are widened exactly),
//   FP32  v_mfma_f32_16x16x4f32,
//   BF16X3 each FP32 operand a = a_hi + a_lo with a_hi = bf16(a),
//          a_lo = bf16(a - a_hi) (round to nearest even), three products
//          hi*hi + hi*lo + lo*hi on v_mfma_f32_16x16x32_bf16.
// Tiles: TILE x TILE per workgroup of 4 wavefronts (2 x 2), each wavefront a
// (TILE/2)^2 block of 16 x 16 MFMA tiles; operands staged through LDS with k
// contiguous.
#include <algorithm>
#include <atomic>

#include "xls_internal.h"

namespace xls {
namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

constexpr int MF_F64 = XLS_PREC_FP64;
constexpr int MF_F32 = XLS_PREC_FP32;
constexpr int MF_BF = XLS_PREC_BF16X3;

__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t nb) {
  const uint32_t xcd = bid & 7u, idx = bid >> 3;
  const uint32_t q = nb >> 3, r = nb & 7u;
  return xcd * q + min(xcd, r) + idx;
}

__device__ __forceinline__ uint16_t bf16_rne_bits(float a) {
  uint32_t u = __float_as_uint(a);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef float f2_t __attribute__((ext_vector_type(2)));
// Split of two FP32 values with the hardware's packed round-to-nearest-even
// conversion: hi = bf16(a), lo = bf16(a - hi); each word holds element 0 in
// its low half (the LDS order of two consecutive bf16 values).  For finite
// values the bits equal bf16_rne_bits'.
__device__ __forceinline__ void split_pair(float a0, float a1, uint32_t& hi, uint32_t& lo) {
  const f2_t a = {a0, a1};
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf2_t));
  const f2_t h = {__uint_as_float(hi << 16), __uint_as_float(hi & 0xFFFF0000u)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(a - h, bf2_t));
}

// ---- per-form traits: LDS element, k per MFMA, operand loads, MFMA --------
template <int MF>
struct Form;

template <>
struct Form<MF_F64> {
  using acc_t = d4_t;
  static constexpr int BK = 16;
  static constexpr int KS = 4;
  static constexpr int PAD = 1;
  using lds_t = double;
  template <typename T>
  __device__ static void put(lds_t* hi, lds_t*, int off, T v) {
    hi[off] = static_cast<double>(v);
  }
  __device__ static void step(acc_t& acc, const lds_t* xh, const lds_t*, const lds_t* yh,
                              const lds_t*, int xrow, int yrow, int stride, int k, int lane) {
    const double a = xh[xrow * stride + k + (lane >> 4)];
    const double b = yh[yrow * stride + k + (lane >> 4)];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
  __device__ static double get(const acc_t& a, int r) { return a[r]; }
  // accumulator element r of a lane holds row (lane/16) + 4r of the 16x16 tile
  __device__ static int orow(int lane, int r) { return (lane >> 4) + 4 * r; }
};

template <>
struct Form<MF_F32> {
  using acc_t = f4_t;
  static constexpr int BK = 16;
  static constexpr int KS = 4;
  static constexpr int PAD = 1;
  using lds_t = float;
  template <typename T>
  __device__ static void put(lds_t* hi, lds_t*, int off, T v) {
    hi[off] = static_cast<float>(v);
  }
  __device__ static void step(acc_t& acc, const lds_t* xh, const lds_t*, const lds_t* yh,
                              const lds_t*, int xrow, int yrow, int stride, int k, int lane) {
    const float a = xh[xrow * stride + k + (lane >> 4)];
    const float b = yh[yrow * stride + k + (lane >> 4)];
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
  }
  __device__ static double get(const acc_t& a, int r) { return a[r]; }
  // accumulator element r of a lane holds row 4(lane/16) + r of the 16x16 tile
  __device__ static int orow(int lane, int r) { return 4 * (lane >> 4) + r; }
};

template <>
struct Form<MF_BF> {
  using acc_t = f4_t;
  static constexpr int BK = 32;
  static constexpr int KS = 32;
  static constexpr int PAD = 8;
  using lds_t = uint16_t;
  template <typename T>
  __device__ static void put(lds_t* hi, lds_t* lo, int off, T v) {
    const float a = static_cast<float>(v);
    const uint16_t h = bf16_rne_bits(a);
    hi[off] = h;
    lo[off] = bf16_rne_bits(a - bf16_bits_to_f32(h));
  }
  __device__ static void step(acc_t& acc, const lds_t* xh, const lds_t* xl, const lds_t* yh,
                              const lds_t* yl, int xrow, int yrow, int stride, int k, int lane) {
    const int ko = k + 8 * (lane >> 4);
    const bf8_t ah = *reinterpret_cast<const bf8_t*>(xh + xrow * stride + ko);
    const bf8_t al = *reinterpret_cast<const bf8_t*>(xl + xrow * stride + ko);
    const bf8_t bh = *reinterpret_cast<const bf8_t*>(yh + yrow * stride + ko);
    const bf8_t bl = *reinterpret_cast<const bf8_t*>(yl + yrow * stride + ko);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
  }
  __device__ static double get(const acc_t& a, int r) { return a[r]; }
  __device__ static int orow(int lane, int r) { return 4 * (lane >> 4) + r; }
};

template <int MF, int TILE>
struct Smem {
  using F = Form<MF>;
  static constexpr int stride = F::BK + F::PAD;
  static constexpr int elems = TILE * stride;                 // one operand, one part
  static constexpr int parts = (MF == MF_BF) ? 2 : 1;
  static constexpr size_t bytes = 2 * parts * elems * sizeof(typename F::lds_t);
};

// C = A^T B partial over one K split.  A: K x M (lda), B: K x N (ldb).
template <typename TIN, int MF, int TILE>
__global__ __launch_bounds__(256) void gemm_tn_kernel(const TIN* __restrict__ A, int64_t lda,
                                                      const TIN* __restrict__ B, int64_t ldb, int M,
                                                      int N, int64_t K, int64_t kchunk, int tm,
                                                      int tn, int sym, double* __restrict__ P) {
  using F = Form<MF>;
  using L = typename F::lds_t;
  constexpr int BK = F::BK, ST = Smem<MF, TILE>::stride, E = Smem<MF, TILE>::elems;
  constexpr int WB = TILE / 32;
  __shared__ __align__(16) L sm[Smem<MF, TILE>::bytes / sizeof(L)];
  L* xh = sm;
  L* yh = sm + E;
  L* xl = (MF == MF_BF) ? sm + 2 * E : nullptr;
  L* yl = (MF == MF_BF) ? sm + 3 * E : nullptr;

  const uint32_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int ntile = sym ? tm * (tm + 1) / 2 : tm * tn;
  const int split = static_cast<int>(lb / ntile);
  int tt = static_cast<int>(lb % ntile);
  int bm, bn;
  if (sym) {  // enumerate upper tiles bm <= bn column by column
    bn = 0;
    while (tt > bn) {
      tt -= bn + 1;
      ++bn;
    }
    bm = tt;
  } else {
    bm = tt % tm;
    bn = tt / tm;
  }
  const int m0 = bm * TILE, n0 = bn * TILE;
  const int64_t kb0 = static_cast<int64_t>(split) * kchunk;
  const int64_t kend = min(K, kb0 + kchunk);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave & 1, wc = wave >> 1;
  typename F::acc_t acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j) acc[i][j] = typename F::acc_t{};

  // A split of a small order is a dozen slabs, each a load latency: two are in
  // flight while a third is multiplied (unconditional loads from clamped
  // addresses; what lies outside is zeroed on its way into LDS).
  constexpr int IT = TILE * BK / 256;
  struct Slab {
    TIN a[IT], b[IT];
  };
  auto load = [&](Slab& v, int64_t kb) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int l = tid + it * 256, r = l / BK;
      const int64_t kk = min(kb + l % BK, K - 1);
      v.a[it] = A[kk + static_cast<int64_t>(min(m0 + r, M - 1)) * lda];
      v.b[it] = B[kk + static_cast<int64_t>(min(n0 + r, N - 1)) * ldb];
    }
  };
  auto slab = [&](Slab& v, int64_t kb) {  // multiplies slab kb and starts slab kb + 2 BK
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int l = tid + it * 256, k = l % BK, r = l / BK;
      const bool kin = kb + k < kend;
      F::put(xh, xl, r * ST + k, kin && m0 + r < M ? v.a[it] : TIN(0));
      F::put(yh, yl, r * ST + k, kin && n0 + r < N ? v.b[it] : TIN(0));
    }
    load(v, kb + 2 * BK);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BK; k += F::KS)
#pragma unroll
      for (int bi = 0; bi < WB; ++bi)
#pragma unroll
        for (int bj = 0; bj < WB; ++bj)
          F::step(acc[bi][bj], xh, xl, yh, yl, wr * (TILE / 2) + bi * 16 + (lane & 15),
                  wc * (TILE / 2) + bj * 16 + (lane & 15), ST, k, lane);
    __syncthreads();
  };
  Slab s0, s1;
  load(s0, kb0);
  load(s1, kb0 + BK);
  for (int64_t kb = kb0; kb < kend; kb += 2 * BK) {
    slab(s0, kb);
    if (kb + BK < kend) slab(s1, kb + BK);
  }
  double* Ps = P + static_cast<int64_t>(split) * M * N;
#pragma unroll
  for (int bi = 0; bi < WB; ++bi)
#pragma unroll
    for (int bj = 0; bj < WB; ++bj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wr * (TILE / 2) + bi * 16 + F::orow(lane, r);
        const int cl = n0 + wc * (TILE / 2) + bj * 16 + (lane & 15);
        if (row < M && cl < N) Ps[row + static_cast<int64_t>(cl) * M] = F::get(acc[bi][bj], r);
      }
}

__global__ void tn_reduce_kernel(const double* __restrict__ P, int splits, int M, int N, int tile,
                                 int sym, int symmetrize, double* __restrict__ C, int64_t ldc) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= static_cast<int64_t>(M) * N) return;
  const int i = static_cast<int>(e % M), j = static_cast<int>(e / M);
  const int64_t MN = static_cast<int64_t>(M) * N;
  auto get = [&](int a, int b) {
    if (sym && (a / tile) > (b / tile)) {
      const int t = a;
      a = b;
      b = t;
    }
    double s = 0.0;
    for (int sp = 0; sp < splits; ++sp) s += P[sp * MN + a + static_cast<int64_t>(b) * M];
    return s;
  };
  double v = get(i, j);
  if (symmetrize) v = 0.5 * (v + get(j, i));
  C[i + static_cast<int64_t>(j) * ldc] = v;
}

// The same reduction for square products that are symmetric (only tiles on
// or above the block diagonal computed) or symmetrized: one block per pair of
// 16 x 16 output tiles (I, J), I <= J, sums the partials of both tiles in
// split order into LDS with coalesced reads, then writes both tiles
// coalesced.  Per element the arithmetic is that of tn_reduce_kernel.  Orders
// of a hundred or two leave a few dozen blocks, each bound by the latency of
// its loads, so kRedU of them are in flight before the first sum, and a tile
// that is its own mirror image or was not computed is not read: 64 splits of
// order 120 54 -> 19 us.
constexpr int kRedT = 16, kRedU = 16;
__global__ __launch_bounds__(256) void tn_reduce_pairs_kernel(const double* __restrict__ P, int splits, int M,
                                                              int tile, int sym, int symmetrize,
                                                              double* __restrict__ C, int64_t ldc, int nt) {
  __shared__ double a[kRedT][kRedT + 1], b[kRedT][kRedT + 1];
  int p = static_cast<int>(blockIdx.x), I = 0;
  while (p >= nt - I) {
    p -= nt - I;
    ++I;
  }
  const int J = I + p;
  const int r = threadIdx.x % kRedT, c = threadIdx.x / kRedT;
  const int64_t MN = static_cast<int64_t>(M) * M;
  const int ai = I * kRedT + r, aj = J * kRedT + c;  // a[r][c] = P(ai, aj)
  const int bi = J * kRedT + r, bj = I * kRedT + c;  // b[r][c] = P(bi, bj)
  const bool va = ai < M && aj < M, vb = bi < M && bj < M;
  const bool mirror = I == J || (sym && J * kRedT / tile > I * kRedT / tile);  // b is a, or not used
  auto sum = [&](const double* src) {
    double s = 0.0;
    int sp = 0;
    for (; sp + kRedU <= splits; sp += kRedU) {
      double v[kRedU];
#pragma unroll
      for (int u = 0; u < kRedU; ++u) v[u] = src[(sp + u) * MN];
#pragma unroll
      for (int u = 0; u < kRedU; ++u) s += v[u];
    }
    if (sp < splits) {  // the rest, also at once
      double v[kRedU];
#pragma unroll
      for (int u = 0; u < kRedU; ++u) v[u] = src[min(sp + u, splits - 1) * MN];
#pragma unroll
      for (int u = 0; u < kRedU; ++u)
        if (sp + u < splits) s += v[u];
    }
    return s;
  };
  const double sa = va ? sum(P + ai + static_cast<int64_t>(aj) * M) : 0.0;
  const double sb = mirror ? sa : (vb ? sum(P + bi + static_cast<int64_t>(bj) * M) : 0.0);
  a[r][c] = sa;
  b[r][c] = sb;
  __syncthreads();
  // element (x, y) of the product: P(x, y), or P(y, x) where a symmetric
  // product kept only the upper block triangle
  {
    const int i = ai, j = aj;  // output (i, j): row in tile I, column in tile J
    const double vij = (sym && i / tile > j / tile) ? b[c][r] : a[r][c];
    const double vji = (sym && j / tile > i / tile) ? a[r][c] : b[c][r];
    if (va) C[i + static_cast<int64_t>(j) * ldc] = symmetrize ? 0.5 * (vij + vji) : vij;
  }
  if (I != J) {
    const int i = bi, j = bj;  // output (i, j): row in tile J, column in tile I
    const double vij = (sym && i / tile > j / tile) ? a[c][r] : b[r][c];
    const double vji = (sym && j / tile > i / tile) ? b[r][c] : a[c][r];
    if (vb) C[i + static_cast<int64_t>(j) * ldc] = symmetrize ? 0.5 * (vij + vji) : vij;
  }
}

void launch_tn_reduce(const double* work, int splits, int M, int N, int tile, int sym, int symmetrize, double* C,
                      int64_t ldc, hipStream_t st) {
  if ((sym || symmetrize) && M == N) {
    const int nt = (M + kRedT - 1) / kRedT;
    const int64_t pairs = static_cast<int64_t>(nt) * (nt + 1) / 2;
    hipLaunchKernelGGL(tn_reduce_pairs_kernel, dim3(static_cast<unsigned>(pairs)), dim3(256), 0, st, work, splits,
                       M, tile, sym, symmetrize, C, ldc, nt);
    XLS_LAUNCH_CHECK("tn_reduce_pairs_kernel");
    return;
  }
  const int64_t tot = static_cast<int64_t>(M) * N;
  hipLaunchKernelGGL(tn_reduce_kernel, dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0, st, work,
                     splits, M, N, tile, sym, symmetrize, C, ldc);
  XLS_LAUNCH_CHECK("tn_reduce_kernel");
}

// C[M x N] = A[M x K] B[K x N]; the MFMA computes the transposed tile so that
// each lane's results run down a column of C (coalesced stores).
template <typename TIN, typename TB, typename TOUT, int MF, int TILE>
__global__ __launch_bounds__(256) void gemm_nn_kernel(const TIN* __restrict__ A, int64_t lda,
                                                      const TB* __restrict__ B, int64_t ldb, int M,
                                                      int N, int K, int tmM, int tnN,
                                                      TOUT* __restrict__ C, int64_t ldc) {
  using F = Form<MF>;
  using L = typename F::lds_t;
  constexpr int BK = F::BK, ST = Smem<MF, TILE>::stride, E = Smem<MF, TILE>::elems;
  constexpr int WB = TILE / 32;
  __shared__ __align__(16) L sm[Smem<MF, TILE>::bytes / sizeof(L)];
  L* ah = sm;  // A tile rows = m
  L* bh = sm + E;  // B tile rows = n
  L* al = (MF == MF_BF) ? sm + 2 * E : nullptr;
  L* bl = (MF == MF_BF) ? sm + 3 * E : nullptr;

  const uint32_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int bn = static_cast<int>(lb % tnN), bm = static_cast<int>(lb / tnN);
  const int m0 = bm * TILE, n0 = bn * TILE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave & 1, wc = wave >> 1;  // wr: n direction, wc: m direction
  typename F::acc_t acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j) acc[i][j] = typename F::acc_t{};

  for (int kb = 0; kb < K; kb += BK) {
#pragma unroll
    for (int it = 0; it < (TILE * BK) / 256; ++it) {
      const int l = tid + it * 256;
      {  // A: coalesced along m
        const int m = l % TILE, k = l / TILE;
        const bool ok = (m0 + m < M) && (kb + k < K);
        const TIN v = ok ? A[(m0 + m) + static_cast<int64_t>(kb + k) * lda] : TIN(0);
        F::put(ah, al, m * ST + k, v);
      }
      {  // B: coalesced along k
        const int k = l % BK, n = l / BK;
        const bool ok = (n0 + n < N) && (kb + k < K);
        const TB v = ok ? B[(kb + k) + static_cast<int64_t>(n0 + n) * ldb] : TB(0);
        F::put(bh, bl, n * ST + k, v);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BK; k += F::KS)
#pragma unroll
      for (int bi = 0; bi < WB; ++bi)
#pragma unroll
        for (int bj = 0; bj < WB; ++bj)
          F::step(acc[bi][bj], bh, bl, ah, al, wr * (TILE / 2) + bi * 16 + (lane & 15),
                  wc * (TILE / 2) + bj * 16 + (lane & 15), ST, k, lane);
    __syncthreads();
  }
#pragma unroll
  for (int bi = 0; bi < WB; ++bi)
#pragma unroll
    for (int bj = 0; bj < WB; ++bj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = n0 + wr * (TILE / 2) + bi * 16 + F::orow(lane, r);
        const int m = m0 + wc * (TILE / 2) + bj * 16 + (lane & 15);
        if (m < M && n < N) C[m + static_cast<int64_t>(n) * ldc] = static_cast<TOUT>(F::get(acc[bi][bj], r));
      }
}

__global__ void split_bf16_kernel(const float* __restrict__ a, uint16_t* __restrict__ hi,
                                  uint16_t* __restrict__ lo, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint16_t h = bf16_rne_bits(a[i]);
  hi[i] = h;
  lo[i] = bf16_rne_bits(a[i] - bf16_bits_to_f32(h));
}

__global__ void d2f_kernel(const double* __restrict__ s, float* __restrict__ d, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) d[i] = static_cast<float>(s[i]);
}


// ---------------------------------------------------------------------------
// Large-tile kernels for the long-K projection and the tall rotation.  Each
// wavefront holds a 4 x 4 block of 16 x 16 MFMA tiles and reuses its operand
// fragments across that block; operands arrive through 16-byte global loads
// staged in registers (the next K slab loads while the current one computes).
// Used when leading dimensions are multiples of the vector width.
// ---------------------------------------------------------------------------
template <int MF>
struct Frag;
template <>
struct Frag<MF_F64> {
  using t = double;
  static constexpr int KS = 4;
  __device__ static t load(const double* h, const double*, int row, int stride, int k, int lane) {
    return h[row * stride + k + (lane >> 4)];
  }
  __device__ static void mma(d4_t& acc, const t& a, const t& b) {
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
};
template <>
struct Frag<MF_F32> {
  using t = float;
  static constexpr int KS = 4;
  __device__ static t load(const float* h, const float*, int row, int stride, int k, int lane) {
    return h[row * stride + k + (lane >> 4)];
  }
  __device__ static void mma(f4_t& acc, const t& a, const t& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
  }
};
// LDS layout of the large-tile BF operands: rows of 32 bf16 (four 16-byte
// chunks) without padding; chunk c of row r sits at position
// c ^ (((r >> 2) ^ (r >> 4)) & 3).  Sixteen consecutive rows then cover all
// 64 banks once for a 16-byte fragment read, eight rows of 64 bytes are
// written in the minimum two passes, and the transposed 32-bit stores of
// the NN kernel (rows 4 j + e) spread over every bank.
__device__ __forceinline__ int bf_off(int r, int k) {
  return r * 32 + (((k >> 3) ^ (((r >> 2) ^ (r >> 4)) & 3)) << 3) + (k & 7);
}

template <>
struct Frag<MF_BF> {
  struct t {
    bf8_t h, l;
  };
  static constexpr int KS = 32;
  // stride is fixed at 32 for this form (bf_off)
  __device__ static t load(const uint16_t* h, const uint16_t* l, int row, int, int k, int lane) {
    const int o = bf_off(row, k + 8 * (lane >> 4));
    return t{*reinterpret_cast<const bf8_t*>(h + o), *reinterpret_cast<const bf8_t*>(l + o)};
  }
  __device__ static void mma(f4_t& acc, const t& a, const t& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, acc, 0, 0, 0);
  }
};

template <int MF>
struct BigLds {
  using L = typename Form<MF>::lds_t;
  static constexpr int BK = (MF == MF_F64) ? 16 : 32;
  // padded rows (16-byte aligned) for FP64/FP32; the BF form swizzles instead (bf_off)
  static constexpr int STRIDE = BK + (MF == MF_BF ? 0 : (MF == MF_F64 ? 2 : 4));
  static constexpr int PARTS = (MF == MF_BF) ? 2 : 1;
};

// Rows of an FP64 or FP32 operand hold one slab of k: 128 bytes, eight 16-byte
// chunks.  Chunk c of row r sits at c ^ ((r >> 1) & 7), so that 16 rows read
// at one chunk, and rows written whole, cover the 64 banks once without
// padding.  Lane group q of a wavefront reads chunk 4 g + q: FP32 rows hold
// k = 16 g + 4 e + q in its element e, so that MFMA step e multiplies four
// consecutive k values as it would from rows in order (the sums keep their
// order), and FP64 rows k = 8 g + 2 q + e.
template <int MF>
__device__ __forceinline__ int chunk_off(int r, int c) {
  constexpr int CH = 16 / sizeof(typename Form<MF>::lds_t), BK = BigLds<MF>::BK;
  static_assert(BK == 8 * CH, "rows of 128 bytes");
  return r * BK + (c ^ ((r >> 1) & 7)) * CH;
}

// Writes the VEC k values k .. k + VEC - 1 of row r into an LDS operand
// (split into bf16 hi/lo for the BF form).
template <int MF, typename TIN, int VEC>
__device__ __forceinline__ void big_put_row(typename Form<MF>::lds_t* h, typename Form<MF>::lds_t* l, int r, int k,
                                            const TIN (&v)[VEC]) {
  if constexpr (MF == MF_BF) {
    static_assert(VEC == 2 || VEC == 4, "pairs of k values");
    const int off = bf_off(r, k);
    uint32_t hp[VEC / 2], lp[VEC / 2];
#pragma unroll
    for (int e = 0; e < VEC / 2; ++e)
      split_pair(static_cast<float>(v[2 * e]), static_cast<float>(v[2 * e + 1]), hp[e], lp[e]);
    if constexpr (VEC == 4) {
      *reinterpret_cast<uint2*>(h + off) = make_uint2(hp[0], hp[1]);
      *reinterpret_cast<uint2*>(l + off) = make_uint2(lp[0], lp[1]);
    } else {
      *reinterpret_cast<uint32_t*>(h + off) = hp[0];
      *reinterpret_cast<uint32_t*>(l + off) = lp[0];
    }
  } else {
    if constexpr (MF == MF_F32) {
      static_assert(VEC == 4, "one k value for each lane group");
#pragma unroll
      for (int q = 0; q < 4; ++q) h[chunk_off<MF>(r, k / 16 * 4 + q) + k % 16 / 4] = v[q];
    } else {
      using V = __attribute__((ext_vector_type(2))) double;
#pragma unroll
      for (int c = 0; c < VEC / 2; ++c)
        *reinterpret_cast<V*>(h + chunk_off<MF>(r, k / 2 + c)) =
            V{static_cast<double>(v[2 * c]), static_cast<double>(v[2 * c + 1])};
    }
  }
}

// Partial C = A^T B over one K split, T x T output tile per workgroup (T =
// 128 or 96): four waves in a 2 x 2 grid, each owning a (T/2) x (T/2)
// sub-tile of NI x NI MFMA blocks of 16 x 16.  The 96 tile covers an order
// of 480 (or any multiple of 96) without padding, and the triangle of a
// symmetric product with less redundant work on its diagonal tiles.
// Bound by the matrix cores.  Two slabs of LDS (one barrier per slab), 16-byte
// fragment reads (a lane group's k values are consecutive: the k order within
// a slab is free as long as both operands share it), columns past the edge
// clamped instead of masked (their sums are not stored) and k masked in the
// last slab only keep other instructions out of the MFMA stream: FP32 K =
// 884736, order 1152 12.2 -> 10.8 ms (121 TFLOP/s of the tiles computed, 106
// before; a library product reaches 154), FP64 K = 262144, order 480 1.47 ->
// 1.19 ms (61 of 73 TFLOP/s), split BF16 there 0.40 -> 0.29 ms.  Writing the
// next slab between the halves of this one was slower (FP32 spills).
template <typename TIN, int MF, int T>
__global__ __launch_bounds__(256, 2) void gemm_tn_big_kernel(const TIN* __restrict__ A, int64_t lda,
                                                          const TIN* __restrict__ B, int64_t ldb, int M,
                                                          int N, int64_t K, int64_t kchunk, int tm, int tn,
                                                          int sym, double* __restrict__ P) {
  using Lc = BigLds<MF>;
  using L = typename Lc::L;
  static_assert(T == 128 || T == 96, "large TN tiles are 128 or 96");
  constexpr int BK = Lc::BK;
  constexpr int WT = T / 2, NI = WT / 16;
  constexpr int VEC = 16 / sizeof(TIN);
  constexpr int PERCOL = BK / VEC;
  static_assert((T * PERCOL) % 256 == 0, "whole loads per thread");
  constexpr int LOADS = T * PERCOL / 256;
  constexpr int CSTEP = 256 / PERCOL;  // columns between a thread's loads
  constexpr int BUF = 2 * Lc::PARTS * T * BK;
  __shared__ __align__(16) L sm[2 * BUF];

  const uint32_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int ntile = sym ? tm * (tm + 1) / 2 : tm * tn;
  const int split = static_cast<int>(lb / ntile);
  int tt = static_cast<int>(lb % ntile);
  int bm, bn;
  if (sym) {
    bn = 0;
    while (tt > bn) {
      tt -= bn + 1;
      ++bn;
    }
    bm = tt;
  } else {
    bm = tt % tm;
    bn = tt / tm;
  }
  const int m0 = bm * T, n0 = bn * T;
  const int64_t kb0 = static_cast<int64_t>(split) * kchunk;
  const int64_t kend = min(K, kb0 + kchunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave & 1, wc = wave >> 1;
  const int c0 = tid / PERCOL, kv = tid % PERCOL * VEC;
  const int nslab = static_cast<int>((kend - kb0 + BK - 1) / BK);
  const int nfull = static_cast<int>((kend - kb0) / BK);

  using V = __attribute__((ext_vector_type(VEC))) TIN;
  const TIN *pa[LOADS], *pb[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int c = c0 + i * CSTEP;
    pa[i] = A + kb0 + kv + static_cast<int64_t>(min(m0 + c, M - 1)) * lda;
    pb[i] = B + kb0 + kv + static_cast<int64_t>(min(n0 + c, N - 1)) * ldb;
  }
  V ra[LOADS], rb[LOADS];
  auto load = [&](int s) {
    if (s < nfull) {
#pragma unroll
      for (int i = 0; i < LOADS; ++i) {
        ra[i] = *reinterpret_cast<const V*>(pa[i]);
        rb[i] = *reinterpret_cast<const V*>(pb[i]);
        pa[i] += BK;
        pb[i] += BK;
      }
    } else {  // the last slab of the last split: k values past K are zero
      const int64_t k = kb0 + static_cast<int64_t>(s) * BK + kv;
#pragma unroll
      for (int i = 0; i < LOADS; ++i) {
        V va{}, vb{};
        if (k < kend) {
          va = *reinterpret_cast<const V*>(pa[i]);
          vb = *reinterpret_cast<const V*>(pb[i]);
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          ra[i][e] = k + e < kend ? va[e] : TIN(0);
          rb[i][e] = k + e < kend ? vb[e] : TIN(0);
        }
      }
    }
  };
  auto store = [&](L* buf) {
    L* xl = (MF == MF_BF) ? buf + 2 * T * BK : nullptr;
    L* yl = (MF == MF_BF) ? buf + 3 * T * BK : nullptr;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int c = c0 + i * CSTEP;
      TIN x[VEC], y[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        x[e] = ra[i][e];
        y[e] = rb[i][e];
      }
      big_put_row<MF, TIN, VEC>(buf, xl, c, kv, x);
      big_put_row<MF, TIN, VEC>(buf + T * BK, yl, c, kv, y);
    }
  };

  typename Form<MF>::acc_t acc[NI][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = typename Form<MF>::acc_t{};
  // The FP32 form (the polish projection) moves its MFMA sums into a
  // second FP32 accumulator every kFlushSteps k-blocks (128 k), so rounding
  // grows over 32 MFMA steps and then over the few hundred flushes of a K
  // split, instead of over thousands of steps in one accumulator.  (FP64
  // registers measured no more accurate at the Ritz level and cost
  // occupancy.)
  constexpr bool FLUSH = (MF == MF_F32);
  constexpr int kFlushSteps = 4;
  float accd[FLUSH ? NI : 1][FLUSH ? NI : 1][4] = {};
  auto flush = [&]() {
    if constexpr (FLUSH) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) accd[i][j][r] += acc[i][j][r];
          acc[i][j] = typename Form<MF>::acc_t{};
        }
    }
  };
  auto compute = [&](const L* buf, int g) {  // half a slab (BF: g = 0 is the whole one)
    const L* x = buf + (wr * WT + (lane & 15)) * BK;
    const L* y = buf + (T + wc * WT + (lane & 15)) * BK;
    if constexpr (MF == MF_BF) {
      if (g == 1) return;
      using FR = Frag<MF>;
      typename FR::t fa[NI], fb[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) fa[i] = FR::load(buf, buf + 2 * T * BK, wr * WT + i * 16 + (lane & 15), BK, 0, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j)
        fb[j] = FR::load(buf + T * BK, buf + 3 * T * BK, wc * WT + j * 16 + (lane & 15), BK, 0, lane);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) FR::mma(acc[i][j], fa[i], fb[j]);
    } else {
      constexpr int CH = 16 / sizeof(L);
      using VL = __attribute__((ext_vector_type(CH))) L;
      const int o = ((4 * g + (lane >> 4)) ^ ((lane >> 1) & 7)) * CH;
      VL fa[NI], fb[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) fa[i] = *reinterpret_cast<const VL*>(x + i * 16 * BK + o);
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[j] = *reinterpret_cast<const VL*>(y + j * 16 * BK + o);
#pragma unroll
      for (int e = 0; e < CH; ++e)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) Frag<MF>::mma(acc[i][j], fa[i][e], fb[j][e]);
    }
  };

  load(0);
  store(sm);
  __syncthreads();
  int cur = 0;
  for (int s = 0; s < nslab; ++s) {
    const bool more = s + 1 < nslab;
    if (more) load(s + 1);
    compute(sm + cur, 0);
    compute(sm + cur, 1);
    if constexpr (FLUSH)
      if (s % kFlushSteps == kFlushSteps - 1) flush();
    cur = BUF - cur;
    if (more) store(sm + cur);
    __syncthreads();
  }
  if constexpr (FLUSH) flush();
  double* Ps = P + static_cast<int64_t>(split) * M * N;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wr * WT + i * 16 + Form<MF>::orow(lane, r);
        const int cl = n0 + wc * WT + j * 16 + (lane & 15);
        const double v = FLUSH ? static_cast<double>(accd[i][j][r]) : Form<MF>::get(acc[i][j], r);
        if (row < M && cl < N) Ps[row + static_cast<int64_t>(cl) * M] = v;
      }
}

// C[M x N] = A[M x K] B[K x N]: 64 rows x TN columns per workgroup (TN =
// 256 or 128), wave w owns columns (TN/4) w .. (TN/4)(w + 1) - 1.  The MFMA x
// operand is B (rows of the accumulator = columns of C), so each lane's
// results for one column are rows m .. m + 15 across lanes (coalesced
// stores).  TB is the B operand as stored: double (FP64), float (FP32) or
// bf16 hi/lo pairs (BF; Bh/Bl).  The split-BF16 form takes it at either
// width; FP64 and FP32 only where a plan forces 256 columns.
template <typename TIN, typename TB, typename TOUT, int MF, int TN>
__global__ __launch_bounds__(256, 2) void gemm_nn_big_kernel(const TIN* __restrict__ A, int64_t lda,
                                                          const TB* __restrict__ Bh, const TB* __restrict__ Bl,
                                                          int64_t ldb, int M, int N, int K, int tnN,
                                                          TOUT* __restrict__ C, int64_t ldc) {
  using Lc = BigLds<MF>;
  using L = typename Lc::L;
  using FR = Frag<MF>;
  static_assert(TN == 256 || TN == 128, "large NN tiles are 256 or 128 columns");
  constexpr int TM = 64, BK = Lc::BK, ST = Lc::STRIDE;
  constexpr int WN = TN / 4, NJ = WN / 16;                // columns and 16-column blocks per wave
  constexpr int VA = 16 / sizeof(TIN);                    // A loads along m
  constexpr int ALOADS = TM * BK / VA / 256;
  constexpr int VB = 16 / sizeof(TB);                     // B loads along k
  static_assert((TN * BK / VB) % 256 == 0, "whole B loads per thread");
  constexpr int BLOADS = TN * BK / VB / 256;
  __shared__ __align__(16) L sm[Lc::PARTS * (TM + TN) * ST];
  L* ah = sm;
  L* bh = sm + TM * ST;
  L* al = (MF == MF_BF) ? sm + (TM + TN) * ST : nullptr;
  L* bl = (MF == MF_BF) ? sm + (TM + TN) * ST + TM * ST : nullptr;

  const uint32_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int bn = static_cast<int>(lb % tnN), bm = static_cast<int>(lb / tnN);
  const int m0 = bm * TM, n0 = bn * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  using VAt = __attribute__((ext_vector_type(VA))) TIN;
  using VBt = __attribute__((ext_vector_type(VB))) TB;
  // The BF form gives each thread the same VA rows at two consecutive k, so
  // that its split stores (hi, lo) pairs of k values as 32-bit words.
  constexpr bool PAIRK = (MF == MF_BF) && ALOADS == 2;
  auto a_k = [&](int i) { return PAIRK ? 2 * (tid / (TM / VA)) + i : (tid + i * 256) / (TM / VA); };
  auto a_m = [&](int i) { return PAIRK ? (tid % (TM / VA)) * VA : ((tid + i * 256) % (TM / VA)) * VA; };
  VAt ra[ALOADS];
  VBt rbh[BLOADS], rbl[BLOADS];
  auto load = [&](int kb) {
#pragma unroll
    for (int i = 0; i < ALOADS; ++i) {
      const int k = a_k(i), mv = a_m(i);
      const bool ok = (kb + k < K) && (m0 + mv < M);
      ra[i] = ok ? *reinterpret_cast<const VAt*>(A + (m0 + mv) + static_cast<int64_t>(kb + k) * lda) : VAt{};
    }
#pragma unroll
    for (int i = 0; i < BLOADS; ++i) {
      const int l = tid + i * 256;
      const int n = l / (BK / VB), kv = (l % (BK / VB)) * VB;
      const bool ok = (n0 + n < N) && (kb + kv < K);
      const int64_t o = (kb + kv) + static_cast<int64_t>(n0 + n) * ldb;
      rbh[i] = ok ? *reinterpret_cast<const VBt*>(Bh + o) : VBt{};
      if constexpr (MF == MF_BF) rbl[i] = ok ? *reinterpret_cast<const VBt*>(Bl + o) : VBt{};
    }
  };
  auto store = [&](int kb) {
    if constexpr (PAIRK) {  // transpose: LDS rows are m, k contiguous
      const int k = a_k(0), mv = a_m(0);
      const int rot = (mv / VA) & (VA - 1);  // lanes write different rows mod 4 per store (bf_off)
#pragma unroll
      for (int e0 = 0; e0 < VA; ++e0) {
        const int e = (e0 + rot) & (VA - 1);
        float x0 = static_cast<float>(ra[0][0]), x1 = static_cast<float>(ra[1][0]);
#pragma unroll
        for (int q = 1; q < VA; ++q)
          if (e == q) {
            x0 = static_cast<float>(ra[0][q]);
            x1 = static_cast<float>(ra[1][q]);
          }
        const bool mi = m0 + mv + e < M;
        uint32_t hp, lp;
        split_pair(mi ? x0 : 0.0f, mi ? x1 : 0.0f, hp, lp);
        const int off = bf_off(mv + e, k);
        *reinterpret_cast<uint32_t*>(ah + off) = hp;
        *reinterpret_cast<uint32_t*>(al + off) = lp;
      }
    }
#pragma unroll
    for (int i = 0; i < (PAIRK ? 0 : ALOADS); ++i) {  // transpose: LDS rows are m, k contiguous
      const int k = a_k(i), mv = a_m(i);
#pragma unroll
      for (int e = 0; e < VA; ++e) {
        const TIN v = (m0 + mv + e < M) ? ra[i][e] : TIN(0);
        if constexpr (MF == MF_BF) {
          const float a = static_cast<float>(v);
          const uint16_t hb = bf16_rne_bits(a);
          ah[(mv + e) * ST + k] = hb;
          al[(mv + e) * ST + k] = bf16_rne_bits(a - bf16_bits_to_f32(hb));
        } else {
          ah[(mv + e) * ST + k] = static_cast<L>(v);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < BLOADS; ++i) {  // LDS rows are n, k contiguous
      const int l = tid + i * 256;
      const int n = l / (BK / VB), kv = (l % (BK / VB)) * VB;
      if constexpr (MF == MF_BF) {  // one 16-byte chunk per part
        VBt vh = rbh[i], vl = rbl[i];
#pragma unroll
        for (int e = 0; e < VB; ++e)
          if (kb + kv + e >= K) {
            vh[e] = 0;
            vl[e] = 0;
          }
        const int off = bf_off(n, kv);
        *reinterpret_cast<VBt*>(bh + off) = vh;
        *reinterpret_cast<VBt*>(bl + off) = vl;
      } else {
#pragma unroll
        for (int e = 0; e < VB; ++e) {
          const bool ke = kb + kv + e < K;
          bh[n * ST + kv + e] = ke ? static_cast<L>(rbh[i][e]) : L(0);
        }
      }
    }
  };

  typename Form<MF>::acc_t acc[NJ][4];
#pragma unroll
  for (int i = 0; i < NJ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = typename Form<MF>::acc_t{};

  load(0);
  for (int kb = 0; kb < K; kb += BK) {
    __syncthreads();
    store(kb);
    __syncthreads();
    if (kb + BK < K) load(kb + BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += FR::KS) {
      typename FR::t fb[NJ], fa[4];
#pragma unroll
      for (int i = 0; i < NJ; ++i) fb[i] = FR::load(bh, bl, wave * WN + i * 16 + (lane & 15), ST, ks, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j) fa[j] = FR::load(ah, al, j * 16 + (lane & 15), ST, ks, lane);
#pragma unroll
      for (int i = 0; i < NJ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) FR::mma(acc[i][j], fb[i], fa[j]);
    }
  }
#pragma unroll
  for (int i = 0; i < NJ; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = n0 + wave * WN + i * 16 + Form<MF>::orow(lane, r);
        const int m = m0 + j * 16 + (lane & 15);
        if (m < M && n < N) C[m + static_cast<int64_t>(n) * ldc] = static_cast<TOUT>(Form<MF>::get(acc[i][j], r));
      }
}

// C[M x N] = A[M x K] B[K x N] for the FP64 and FP32 forms: TM rows (128, or 64
// where the grid would leave compute units idle) x TN columns (128 or 96) per
// workgroup, four waves in a 2 x 2 grid.  The x operand is B, so a lane's
// results for one column are rows of C.  A stays as it lies in memory, [k][m]:
// a lane reads MW consecutive rows at once and these go to MW different MFMA
// blocks, which makes the block's rows every MW-th one and its stores MW
// values wide.  B rows lie in LDS like the operands of A^T B (FP32 B comes in
// that k order, its rows past K zero), with the same two slabs and edge rules.  Bound by the matrix cores: FP32
// 884736 x 1152 x 1152 20.7 -> 18.4 ms (128 TFLOP/s; 64 x 128 tiles stored
// transposed before; 17.3 with k in chunk order, which sums differently), FP64 262144 x 480 x 480 2.32 -> 1.86 ms (65 of the 73
// TFLOP/s that a library product reaches).
template <typename TIN, typename TOUT, int MF, int TM, int TN>
__global__ __launch_bounds__(256, 2) void gemm_nn_wide_kernel(const TIN* __restrict__ A, int64_t lda,
                                                              const typename Form<MF>::lds_t* __restrict__ B,
                                                              int64_t ldb, int M, int N, int K, int tnN,
                                                              TOUT* __restrict__ C, int64_t ldc, int vecc) {
  using L = typename Form<MF>::lds_t;
  constexpr int BK = BigLds<MF>::BK, CH = 16 / sizeof(L);
  constexpr int MB = TM / 32, NB = TN / 32;             // 16 x 16 blocks of a wave
  constexpr int MW = MB < CH ? MB : CH, PR = MB / MW;   // rows per A read, reads per k
  constexpr int VA = 16 / sizeof(TIN);
  constexpr int APER = TM / VA, ALOADS = BK * APER / 256, ASTEP = 256 / APER;
  constexpr int BPER = BK / CH, BLOADS = TN * BPER / 256, BSTEP = 256 / BPER;
  static_assert(ALOADS * 256 == BK * APER && BLOADS * 256 == TN * BPER, "whole loads per thread");
  constexpr int BUF = (TM + TN) * BK;
  __shared__ __align__(16) L sm[2 * BUF];

  const uint32_t lb = xcd_remap(blockIdx.x, gridDim.x);
  const int bn = static_cast<int>(lb % tnN), bm = static_cast<int>(lb / tnN);
  const int m0 = bm * TM, n0 = bn * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave & 1) * (TM / 2), wn = (wave >> 1) * (TN / 2);
  const int ak = tid / APER, am = tid % APER * VA;
  const int bc = tid / BPER, bk = tid % BPER * CH;
  const int nslab = (K + BK - 1) / BK, nfull = K / BK;

  using VAt = __attribute__((ext_vector_type(VA))) TIN;
  using VL = __attribute__((ext_vector_type(CH))) L;
  using VM = __attribute__((ext_vector_type(MW))) L;
  const TIN* pa = A + min(m0 + am, (M - 1) / VA * VA) + static_cast<int64_t>(ak) * lda;
  const L* pb[BLOADS];
#pragma unroll
  for (int i = 0; i < BLOADS; ++i) pb[i] = B + bk + static_cast<int64_t>(min(n0 + bc + i * BSTEP, N - 1)) * ldb;
  VAt ra[ALOADS];
  VL rb[BLOADS];
  auto load = [&](int s) {
    if (s < nfull) {
#pragma unroll
      for (int i = 0; i < ALOADS; ++i) ra[i] = *reinterpret_cast<const VAt*>(pa + static_cast<int64_t>(i * ASTEP) * lda);
#pragma unroll
      for (int i = 0; i < BLOADS; ++i) rb[i] = *reinterpret_cast<const VL*>(pb[i]);
    } else {  // the last slab: k values past K are zero
#pragma unroll
      for (int i = 0; i < ALOADS; ++i) {
        ra[i] = VAt{};
        if (s * BK + ak + i * ASTEP < K) ra[i] = *reinterpret_cast<const VAt*>(pa + static_cast<int64_t>(i * ASTEP) * lda);
      }
      const int k = s * BK + bk;
#pragma unroll
      for (int i = 0; i < BLOADS; ++i) {
        VL v{};
        if (k < (MF == MF_F32 ? ldb : K)) v = *reinterpret_cast<const VL*>(pb[i]);
#pragma unroll
        for (int e = 0; e < CH; ++e) rb[i][e] = MF == MF_F32 || k + e < K ? v[e] : L(0);
      }
    }
    pa += static_cast<int64_t>(BK) * lda;
#pragma unroll
    for (int i = 0; i < BLOADS; ++i) pb[i] += BK;
  };
  auto store = [&](L* buf) {
#pragma unroll
    for (int i = 0; i < ALOADS; ++i)
#pragma unroll
      for (int c = 0; c < VA / CH; ++c) {
        VL w;
#pragma unroll
        for (int e = 0; e < CH; ++e) w[e] = static_cast<L>(ra[i][c * CH + e]);
        *reinterpret_cast<VL*>(buf + (ak + i * ASTEP) * TM + am + c * CH) = w;
      }
#pragma unroll
    for (int i = 0; i < BLOADS; ++i)
      *reinterpret_cast<VL*>(buf + TM * BK + chunk_off<MF>(bc + i * BSTEP, bk / CH)) = rb[i];
  };

  typename Form<MF>::acc_t acc[NB][MB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = typename Form<MF>::acc_t{};
  auto compute = [&](const L* buf, int g) {  // half a slab
    const L* x = buf + TM * BK + (wn + (lane & 15)) * BK;
    const L* y = buf + wm + (lane & 15) * MW;
    const int q = lane >> 4, o = ((4 * g + q) ^ ((lane >> 1) & 7)) * CH;
    VL fb[NB];
    VM fa[CH][PR];
#pragma unroll
    for (int i = 0; i < NB; ++i) fb[i] = *reinterpret_cast<const VL*>(x + i * 16 * BK + o);
#pragma unroll
    for (int e = 0; e < CH; ++e)
#pragma unroll
      for (int p = 0; p < PR; ++p) {
        const int k = MF == MF_F32 ? 16 * g + 4 * e + q : 8 * g + 2 * q + e;
        fa[e][p] = *reinterpret_cast<const VM*>(y + k * TM + p * 16 * MW);
      }
#pragma unroll
    for (int e = 0; e < CH; ++e)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) Frag<MF>::mma(acc[i][j], fb[i][e], fa[e][j / MW][j % MW]);
  };

  load(0);
  store(sm);
  __syncthreads();
  int cur = 0;
  for (int s = 0; s < nslab; ++s) {
    const bool more = s + 1 < nslab;
    if (more) load(s + 1);
    compute(sm + cur, 0);
    compute(sm + cur, 1);
    cur = BUF - cur;
    if (more) store(sm + cur);
    __syncthreads();
  }
  using VC = __attribute__((ext_vector_type(MW))) TOUT;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = n0 + wn + i * 16 + Form<MF>::orow(lane, r);
      if (n >= N) continue;
#pragma unroll
      for (int p = 0; p < PR; ++p) {
        const int m = m0 + wm + p * 16 * MW + (lane & 15) * MW;
        TOUT* dst = C + m + static_cast<int64_t>(n) * ldc;
        if (vecc && m + MW <= M) {
          VC v;
#pragma unroll
          for (int w = 0; w < MW; ++w) v[w] = static_cast<TOUT>(Form<MF>::get(acc[i][p * MW + w], r));
          *reinterpret_cast<VC*>(dst) = v;
        } else {
#pragma unroll
          for (int w = 0; w < MW; ++w)
            if (m + w < M) dst[w] = static_cast<TOUT>(Form<MF>::get(acc[i][p * MW + w], r));
        }
      }
    }
}

// The rotation matrix B (rows x cols, leading dimension lds) copied with a
// leading dimension ldd >= rows padded to the kernels' 16-byte k loads; the
// padding rows are zero.  FP64 copy, FP32 rounding, or bf16 hi/lo split.
__global__ void pad_f64_kernel(const double* __restrict__ s, int64_t lds, double* __restrict__ d, int64_t ldd,
                               int64_t rows, int64_t cols) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= ldd * cols) return;
  const int64_t r = i % ldd, c = i / ldd;
  d[i] = r < rows ? s[r + c * lds] : 0.0;
}
// (chunked: rows in the order of chunk_off's FP32 rows, ldd a multiple of 16)
__global__ void pad_f32_kernel(const double* __restrict__ s, int64_t lds, float* __restrict__ d, int64_t ldd,
                               int64_t rows, int64_t cols, int chunked) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= ldd * cols) return;
  const int64_t p = i % ldd, c = i / ldd;
  const int64_t r = chunked ? p / 16 * 16 + 4 * (p % 4) + p % 16 / 4 : p;
  d[i] = r < rows ? static_cast<float>(s[r + c * lds]) : 0.0f;
}
__global__ void split_bf16_from_f64_kernel(const double* __restrict__ s, int64_t lds, uint16_t* __restrict__ hi,
                                           uint16_t* __restrict__ lo, int64_t ldd, int64_t rows, int64_t cols) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= ldd * cols) return;
  const int64_t r = i % ldd, c = i / ldd;
  const float a = r < rows ? static_cast<float>(s[r + c * lds]) : 0.0f;
  const uint16_t h = bf16_rne_bits(a);
  hi[i] = h;
  lo[i] = bf16_rne_bits(a - bf16_bits_to_f32(h));
}

constexpr int kTile = 64;

// compute units of the current device (cached per device)
int device_cus() {
  static std::atomic<int> cached[64];
  int dev = 0;
  XLS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) dev = 0;
  int c = cached[dev].load(std::memory_order_relaxed);
  if (c == 0) {
    XLS_HIP(hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev));
    c = std::max(1, c);
    cached[dev].store(c, std::memory_order_relaxed);
  }
  return c;
}

int planned_splits(int def, const GemmPlan& plan);

int choose_splits(int tiles, int64_t K, int bk, int M, int N, size_t work_elems, const GemmPlan& plan) {
  // aim for ~2048 workgroups; each split must keep >= 8 k-blocks
  int s = planned_splits(std::max(1, 2048 / std::max(1, tiles)), plan);
  const int64_t kblocks = (K + bk - 1) / bk;
  s = static_cast<int>(std::min<int64_t>(s, std::max<int64_t>(1, kblocks / 8)));
  const size_t per = static_cast<size_t>(M) * N;
  if (per > 0) s = static_cast<int>(std::min<size_t>(s, std::max<size_t>(1, work_elems / per)));
  return std::max(1, s);
}

template <typename T>
bool aligned16(const T* p) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}

// Split count of a plan: the default rule's count scaled by split_scale / 2.
int planned_splits(int def, const GemmPlan& plan) {
  return plan.split_scale > 0 ? std::max(1, def * plan.split_scale / 2) : def;
}

// K splits of the large TN kernel with tile edge T: about as many workgroups
// as are resident at once (2 per CU at edge 128, 3 at edge 96: its smaller
// accumulator tile leaves room for a third), so that symmetric products
// (fewer tiles) get more splits; >= 16 K slabs each.  The FP32 form counts
// splits for tn_area_edge, whichever edge then runs: its sums are as sensitive to
// their order as to anything else, and so keep it.
struct TnCut {
  int ntile, splits;
  int64_t kchunk;
};
int tn_tiles(int M, int N, int sym, int T) {
  const int tm = (M + T - 1) / T, tn = (N + T - 1) / T;
  return sym ? tm * (tm + 1) / 2 : tm * tn;
}
// the edge that issues 10 % less padded and redundant area, 128 if neither does
int tn_area_edge(int M, int N, int sym) {
  return 10 * int64_t{96 * 96} * tn_tiles(M, N, sym, 96) < 9 * int64_t{128 * 128} * tn_tiles(M, N, sym, 128) ? 96 : 128;
}
TnCut tn_cut(int M, int N, int64_t K, int sym, int T, bool f32, int bk, size_t work_elems, const GemmPlan& plan) {
  TnCut c;
  c.ntile = tn_tiles(M, N, sym, T);
  const int ts = f32 && plan.tile_tn == 0 ? tn_area_edge(M, N, sym) : T;
  const int resident = (ts == 96) ? 3 : 2;
  int splits = planned_splits(std::max(1, resident * device_cus() / tn_tiles(M, N, sym, ts)), plan);
  splits = static_cast<int>(std::min<int64_t>(splits, std::max<int64_t>(1, K / (16 * bk))));
  const size_t per = static_cast<size_t>(M) * N;
  splits = static_cast<int>(std::min<size_t>(splits, std::max<size_t>(1, work_elems / per)));
  c.kchunk = (K + splits - 1) / splits;
  c.kchunk = ((c.kchunk + bk - 1) / bk) * bk;
  c.splits = static_cast<int>((K + c.kchunk - 1) / c.kchunk);
  return c;
}

// Large-tile edge (unless the plan forces one): the one whose busiest compute
// unit has less to multiply, tile area x k of a split x workgroups on it; a
// lone workgroup there runs about a tenth slower for want of a second to
// cover its barriers, and the smaller tile about a twentieth for its LDS reads.  Measured ratios 96 / 128 follow it: 480 of FP64 0.85
// (0.89 by the rule), 300 of FP32 0.86 (0.89), 1200 of FP32 1.01 (1.00), 1152
// of FP32 1.12 (1.08), 200 of FP64 1.07 (1.07), 120 of FP64 0.73 (0.59).
// Split BF16 takes the edge by area: only entries of diagonal tiles of H_s are
// averaged with their transposes, its two triangles differ by more than the
// others', and the smaller tile leaves its H_s up to 1 % further off (order 100,
// K = 35,904: 9.94e-7 against 9.85e-7) for at most 8 us.
template <int MF>
int tn_tile_edge(int M, int N, int64_t K, int sym, int bk, size_t work_elems, const GemmPlan& plan) {
  if (plan.tile_tn == 2) return 128;
  if (plan.tile_tn == 3) return 96;
  if (MF == MF_BF) return tn_area_edge(M, N, sym);
  const auto cost = [&](int T) {
    const TnCut c = tn_cut(M, N, K, sym, T, MF == MF_F32, bk, work_elems, plan);
    const int64_t nb = static_cast<int64_t>(c.ntile) * c.splits, cus = device_cus();
    return static_cast<double>(T) * T * c.kchunk * ((nb + cus - 1) / cus) * (nb <= cus ? 1.1 : 1.0) *
           (T == 96 ? 1.05 : 1.0);
  };
  return cost(96) < cost(128) ? 96 : 128;
}

template <typename TIN, int MF, int T>
void tn_big_launch(const TIN* A, int64_t lda, const TIN* B, int64_t ldb, int M, int N, int64_t K, double* C,
                   int64_t ldc, int sym, int symmetrize, double* work, size_t work_elems, hipStream_t st,
                   const GemmPlan& plan) {
  const int tm = (M + T - 1) / T, tn = (N + T - 1) / T;
  const TnCut c = tn_cut(M, N, K, sym, T, MF == MF_F32, BigLds<MF>::BK, work_elems, plan);
  const int64_t nb = static_cast<int64_t>(c.ntile) * c.splits;
  if (nb > 0x7fffffff) fail(XLS_ERR_INVALID_ARG, "gemm_tn grid too large");
  hipLaunchKernelGGL((gemm_tn_big_kernel<TIN, MF, T>), dim3(static_cast<unsigned>(nb)), dim3(256), 0, st, A,
                     lda, B, ldb, M, N, K, c.kchunk, tm, tn, sym, work);
  XLS_LAUNCH_CHECK("gemm_tn_big_kernel");
  launch_tn_reduce(work, c.splits, M, N, T, sym, symmetrize, C, ldc, st);
}

template <typename TIN, int MF>
void tn_dispatch(const TIN* A, int64_t lda, const TIN* B, int64_t ldb, int M, int N, int64_t K,
                 double* C, int64_t ldc, int sym, int symmetrize, double* work, size_t work_elems,
                 hipStream_t st, const GemmPlan& plan) {
  constexpr int VEC = 16 / sizeof(TIN);
  if (plan.tile_tn != 1 && M >= 64 && N >= 64 && lda % VEC == 0 && ldb % VEC == 0 && K <= lda && K <= ldb &&
      aligned16(A) && aligned16(B)) {
    // the 96 edge needs whole 16-byte loads per thread (not the FP64
    // products of FP32 blocks: 4 loads per 16-wide k slab and row)
    constexpr bool k96 = (96 * (BigLds<MF>::BK / VEC)) % 256 == 0;
    if constexpr (k96) {
      if (tn_tile_edge<MF>(M, N, K, sym, BigLds<MF>::BK, work_elems, plan) == 96) {
        tn_big_launch<TIN, MF, 96>(A, lda, B, ldb, M, N, K, C, ldc, sym, symmetrize, work, work_elems, st, plan);
        return;
      }
    }
    tn_big_launch<TIN, MF, 128>(A, lda, B, ldb, M, N, K, C, ldc, sym, symmetrize, work, work_elems, st, plan);
    return;
  }
  const int tm = (M + kTile - 1) / kTile, tn = (N + kTile - 1) / kTile;
  const int ntile = sym ? tm * (tm + 1) / 2 : tm * tn;
  const int bk = Form<MF>::BK;
  const int splits = choose_splits(ntile, K, bk, M, N, work_elems, plan);
  int64_t kchunk = (K + splits - 1) / splits;
  kchunk = ((kchunk + bk - 1) / bk) * bk;
  const int real_splits = static_cast<int>((K + kchunk - 1) / kchunk);
  const int64_t nb = static_cast<int64_t>(ntile) * real_splits;
  if (nb > 0x7fffffff) fail(XLS_ERR_INVALID_ARG, "gemm_tn grid too large");
  hipLaunchKernelGGL((gemm_tn_kernel<TIN, MF, kTile>), dim3(static_cast<unsigned>(nb)), dim3(256), 0,
                     st, A, lda, B, ldb, M, N, K, kchunk, tm, tn, sym, work);
  XLS_LAUNCH_CHECK("gemm_tn_kernel");
  launch_tn_reduce(work, real_splits, M, N, kTile, sym, symmetrize, C, ldc, st);
}

}  // namespace

size_t nn_work_doubles(int K, int N) {
  return static_cast<size_t>((static_cast<int64_t>(K) + 7) / 8 * 8) * static_cast<size_t>(N);
}

size_t gemm_tn_work_elems(int M, int N, int64_t K) {
  // room for every split either kernel takes (each split keeps >= 8 k-blocks
  // of >= 16, so at most K/128 of them; at most 64), capped at 32 Mi doubles
  // (256 MB)
  const size_t per = static_cast<size_t>(M) * N;
  const size_t splits = static_cast<size_t>(std::min<int64_t>(64, std::max<int64_t>(1, K / 128)));
  return std::max<size_t>(per, std::min<size_t>(splits * per, static_cast<size_t>(32) << 20));
}

template <typename TS>
void gemm_tn(int prec, const TS* A, int64_t lda, const TS* B, int64_t ldb, int M, int N, int64_t K,
             double* C, int64_t ldc, int sym, int symmetrize, double* work, size_t work_elems,
             hipStream_t st, const GemmPlan& plan) {
  if (M <= 0 || N <= 0) return;
  if (work_elems < static_cast<size_t>(M) * N) fail(XLS_ERR_INVALID_ARG, "gemm_tn workspace too small");
  if constexpr (std::is_same<TS, double>::value) {
    if (prec != MF_F64) fail(XLS_ERR_INVALID_ARG, "FP64 blocks use FP64 GEMMs");
    tn_dispatch<double, MF_F64>(A, lda, B, ldb, M, N, K, C, ldc, sym, symmetrize, work, work_elems, st, plan);
  } else {
    if (prec == MF_F64)
      tn_dispatch<float, MF_F64>(A, lda, B, ldb, M, N, K, C, ldc, sym, symmetrize, work, work_elems, st, plan);
    else if (prec == MF_F32)
      tn_dispatch<float, MF_F32>(A, lda, B, ldb, M, N, K, C, ldc, sym, symmetrize, work, work_elems, st, plan);
    else if (prec == MF_BF)
      tn_dispatch<float, MF_BF>(A, lda, B, ldb, M, N, K, C, ldc, sym, symmetrize, work, work_elems, st, plan);
    else
      fail(XLS_ERR_INVALID_ARG, "unknown GEMM precision");
  }
}

// Large-tile rotation of the FP64 and FP32 forms: B as the kernel's operand
// type, leading dimension a multiple of its 16-byte loads.
template <typename TS, int MF>
void nn_wide_launch(const TS* A, int64_t lda, const typename Form<MF>::lds_t* B, int64_t ldb, int M, int N, int K,
                    TS* C, int64_t ldc, hipStream_t st, const GemmPlan& plan) {
  const auto tiles = [](int n, int t) { return (n + t - 1) / t; };
  // 96 columns where they pad N less than 128 do (a forced 128 through the plan otherwise)
  const int tn = (plan.tile_nn != 3 && tiles(N, 96) * 96 < tiles(N, 128) * 128) ? 96 : 128;
  // 64 rows where 128 would leave fewer than two workgroups per CU
  const int64_t nb128 = static_cast<int64_t>(tiles(M, 128)) * tiles(N, tn);
  const int tm = nb128 < 2 * device_cus() ? 64 : 128;
  const int vecc = ldc % 4 == 0 && aligned16(C);
  const int tnN = tiles(N, tn);
  const dim3 grid(static_cast<unsigned>(static_cast<int64_t>(tiles(M, tm)) * tnN));
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, A, lda, B, ldb, M, N, K, tnN, C, ldc, vecc);
  };
  if (tm == 128 && tn == 128) go(gemm_nn_wide_kernel<TS, TS, MF, 128, 128>);
  else if (tm == 128) go(gemm_nn_wide_kernel<TS, TS, MF, 128, 96>);
  else if (tn == 128) go(gemm_nn_wide_kernel<TS, TS, MF, 64, 128>);
  else go(gemm_nn_wide_kernel<TS, TS, MF, 64, 96>);
}

// Large-tile rotation with TN-column tiles; false when the shapes or
// alignment do not allow it.
template <typename TS, int TN>
bool nn_big_t(int prec, const TS* A, int64_t lda, const double* B, int64_t ldb, int M, int N, int K, TS* C,
              int64_t ldc, void* bwork, hipStream_t st, const GemmPlan& plan) {
  constexpr int VA = 16 / sizeof(TS);
  if (M < 64 || N < 64 || lda % VA != 0 || !aligned16(A) || M > lda || K > ldb) return false;
  const bool have_work = bwork != nullptr && aligned16(bwork);
  const int tnN = (N + TN - 1) / TN;
  const int64_t nb = static_cast<int64_t>((M + 63) / 64) * tnN;
  if (nb > 0x7fffffff) return false;
  const dim3 grid(static_cast<unsigned>(nb));
  // B goes through bwork with its leading dimension padded to 8 rows
  // (bwork holds nn_work_elems(K, N) doubles)
  const int64_t ldp = (static_cast<int64_t>(K) + 7) / 8 * 8;
  const int64_t nbv = ldp * static_cast<int64_t>(N);
  const unsigned pgrid = static_cast<unsigned>((nbv + 255) / 256);
  if (prec == MF_F64) {
    const double* Bd = B;
    int64_t ldbd = ldb;
    if (ldb % 2 != 0 || !aligned16(B)) {
      if (!have_work) return false;
      double* Bp = static_cast<double*>(bwork);
      hipLaunchKernelGGL(pad_f64_kernel, dim3(pgrid), dim3(256), 0, st, B, ldb, Bp, ldp, K, N);
      Bd = Bp;
      ldbd = ldp;
    }
    if constexpr (TN == 128)
      nn_wide_launch<TS, MF_F64>(A, lda, Bd, ldbd, M, N, K, C, ldc, st, plan);
    else
      hipLaunchKernelGGL((gemm_nn_big_kernel<TS, double, TS, MF_F64, TN>), grid, dim3(256), 0, st, A, lda, Bd,
                         static_cast<const double*>(nullptr), ldbd, M, N, K, tnN, C, ldc);
  } else if constexpr (std::is_same<TS, float>::value) {
    if (!have_work) return false;
    if (prec == MF_F32) {
      float* Bf = static_cast<float*>(bwork);
      // 16-row chunks of FP32 need no more room than 8-row chunks of FP64
      const int64_t ldf = TN == 128 ? (static_cast<int64_t>(K) + 15) / 16 * 16 : ldp;
      hipLaunchKernelGGL(pad_f32_kernel, dim3(static_cast<unsigned>((ldf * N + 255) / 256)), dim3(256), 0, st, B, ldb,
                         Bf, ldf, K, N, TN == 128 ? 1 : 0);
      if constexpr (TN == 128)
        nn_wide_launch<float, MF_F32>(A, lda, Bf, ldf, M, N, K, C, ldc, st, plan);
      else
        hipLaunchKernelGGL((gemm_nn_big_kernel<float, float, float, MF_F32, TN>), grid, dim3(256), 0, st, A, lda,
                           Bf, static_cast<const float*>(nullptr), ldf, M, N, K, tnN, C, ldc);
    } else if (prec == MF_BF) {
      // the rotation matrix is split into bf16 hi/lo once (same bytes as its FP32 copy)
      uint16_t* bh = static_cast<uint16_t*>(bwork);
      uint16_t* bl = bh + nbv;
      hipLaunchKernelGGL(split_bf16_from_f64_kernel, dim3(pgrid), dim3(256), 0, st, B, ldb, bh, bl, ldp, K, N);
      hipLaunchKernelGGL((gemm_nn_big_kernel<float, uint16_t, float, MF_BF, TN>), grid, dim3(256), 0, st, A, lda, bh, bl,
                         ldp, M, N, K, tnN, C, ldc);
    } else {
      return false;
    }
  } else {
    return false;
  }
  XLS_LAUNCH_CHECK("gemm_nn_big_kernel");
  return true;
}

template <typename TS>
bool nn_big(int prec, const TS* A, int64_t lda, const double* B, int64_t ldb, int M, int N, int K, TS* C,
            int64_t ldc, void* bwork, hipStream_t st, const GemmPlan& plan) {
  // 128 columns unless the plan forces 256, which pads N no less and measured
  // 2-5 % slower where both pad alike (N = 480)
  if (plan.tile_nn != 2) return nn_big_t<TS, 128>(prec, A, lda, B, ldb, M, N, K, C, ldc, bwork, st, plan);
  return nn_big_t<TS, 256>(prec, A, lda, B, ldb, M, N, K, C, ldc, bwork, st, plan);
}

template <typename TS>
void gemm_nn(int prec, const TS* A, int64_t lda, const double* B, int64_t ldb, int M, int N, int K,
             TS* C, int64_t ldc, void* bwork, hipStream_t st, const GemmPlan& plan) {
  if (M <= 0 || N <= 0) return;
  if (plan.tile_nn != 1 && nn_big<TS>(prec, A, lda, B, ldb, M, N, K, C, ldc, bwork, st, plan)) return;
  const int tmM = (M + kTile - 1) / kTile, tnN = (N + kTile - 1) / kTile;
  const int64_t nb = static_cast<int64_t>(tmM) * tnN;
  if (nb > 0x7fffffff) fail(XLS_ERR_INVALID_ARG, "gemm_nn grid too large");
  const dim3 grid(static_cast<unsigned>(nb));
  if constexpr (std::is_same<TS, double>::value) {
    if (prec != MF_F64) fail(XLS_ERR_INVALID_ARG, "FP64 blocks use FP64 GEMMs");
    hipLaunchKernelGGL((gemm_nn_kernel<double, double, double, MF_F64, kTile>), grid, dim3(256), 0, st,
                       A, lda, B, ldb, M, N, K, tmM, tnN, C, ldc);
  } else {
    if (prec == MF_F64) {
      hipLaunchKernelGGL((gemm_nn_kernel<float, double, float, MF_F64, kTile>), grid, dim3(256), 0, st,
                         A, lda, B, ldb, M, N, K, tmM, tnN, C, ldc);
    } else {
      // the rotation matrix is rounded to FP32 once, then fed like the block
      float* Bf = static_cast<float*>(bwork);
      const int64_t nbv = ldb * static_cast<int64_t>(N);
      hipLaunchKernelGGL(d2f_kernel, dim3(static_cast<unsigned>((nbv + 255) / 256)), dim3(256), 0, st, B, Bf,
                         nbv);
      if (prec == MF_F32)
        hipLaunchKernelGGL((gemm_nn_kernel<float, float, float, MF_F32, kTile>), grid, dim3(256), 0, st,
                           A, lda, Bf, ldb, M, N, K, tmM, tnN, C, ldc);
      else if (prec == MF_BF)
        hipLaunchKernelGGL((gemm_nn_kernel<float, float, float, MF_BF, kTile>), grid, dim3(256), 0, st,
                           A, lda, Bf, ldb, M, N, K, tmM, tnN, C, ldc);
      else
        fail(XLS_ERR_INVALID_ARG, "unknown GEMM precision");
    }
  }
  XLS_LAUNCH_CHECK("gemm_nn_kernel");
}

void split_bf16_device(const float* a, uint16_t* hi, uint16_t* lo, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(split_bf16_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st,
                     a, hi, lo, n);
  XLS_LAUNCH_CHECK("split_bf16_kernel");
}

template void gemm_tn<double>(int, const double*, int64_t, const double*, int64_t, int, int, int64_t,
                              double*, int64_t, int, int, double*, size_t, hipStream_t, const GemmPlan&);
template void gemm_tn<float>(int, const float*, int64_t, const float*, int64_t, int, int, int64_t,
                             double*, int64_t, int, int, double*, size_t, hipStream_t, const GemmPlan&);
template void gemm_nn<double>(int, const double*, int64_t, const double*, int64_t, int, int, int,
                              double*, int64_t, void*, hipStream_t, const GemmPlan&);
template void gemm_nn<float>(int, const float*, int64_t, const double*, int64_t, int, int, int, float*,
                             int64_t, void*, hipStream_t, const GemmPlan&);

}  // namespace xls
