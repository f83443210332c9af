// Electrostatic Poisson solve (Sec. IV Poisson equation; Sec. V-B.1
// structured-multigrid-preconditioned CG): A phi = 4 pi f with A = -L the
// 12th-order FD Laplacian (zero Dirichlet or periodic), CG in FP64,
// preconditioned by one FP32 V-cycle whose finest level is the 7-point
// Laplacian applied matrix-free and whose coarse levels are the Galerkin
// operators P^T A P of trilinear prolongation.  On a uniform grid with exact
// coarsening those are one 27-point stencil per level, computed once on the
// host from the fine stencil; every level is applied matrix-free.
//
// Coarsening: zero Dirichlet n -> (n - 1)/2 (coarse point I on fine 2I + 1),
// periodic n -> n/2 (coarse I on fine 2I), while every axis coarsens exactly
// to at least 3 (4) points.  Smoothing: damped Jacobi (omega = 2/3), nu
// sweeps before and after the coarse correction, nu_c sweeps from zero on the
// coarsest level; zero start makes the V-cycle symmetric.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "xls_handle.h"

using namespace xls;

namespace {

constexpr int R12 = 6;  // half-width of the 12th-order Laplacian
constexpr int Q12 = 2 * R12 + 1;
constexpr float kOmega = 2.0f / 3.0f;
constexpr int kNu = 2, kNuCoarse = 10;

inline unsigned nblk(int64_t n, int b) { return static_cast<unsigned>((n + b - 1) / b); }

struct Grid {
  int nx, ny, nz;
  int periodic;
};

__device__ __forceinline__ int wrap(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

// Block id -> logical id such that consecutive logical ids land on the same
// XCD (workgroups are dealt round-robin to 8): neighbouring tiles share their
// halo rows in that XCD's L2.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t bid, uint32_t nb) {
  const uint32_t xcd = bid & 7u, idx = bid >> 3;
  const uint32_t q = nb >> 3, r = nb & 7u;
  return xcd * q + min(xcd, r) + idx;
}

// Sum over a 256-thread workgroup (fixed order); valid in thread 0.
__device__ __forceinline__ double block_total(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Workgroup barrier that waits for LDS traffic only (see the filter stencil):
// the next plane's global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __asm__ __volatile__("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  __asm__ __volatile__("" ::: "memory");
}

// Tile of a marching kernel: x0, y0 of the xy tile and the planes [z0, z1).
struct March {
  int nbx, nby, tz;
};
struct Tile {
  int bx, by, z0, z1;
};
__device__ __forceinline__ Tile march_tile(const March& m, int nz) {
  const uint32_t l = xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t per = static_cast<uint32_t>(m.nbx) * m.nby;
  const int zt = static_cast<int>(l / per);
  const uint32_t rem = l % per;
  const int z0 = zt * m.tz;
  return Tile{static_cast<int>(rem % m.nbx), static_cast<int>(rem / m.nbx), z0, min(z0 + m.tz, nz)};
}

// Coordinate along an axis wrapped (periodic) or clamped into the grid; in is
// false beyond a Dirichlet face (the caller's value is then zero).
__device__ __forceinline__ int axis(int i, int n, int periodic, bool& in) {
  if (periodic) {
    if (i < 0 || i >= n) i = wrap(i, n);
    return i;
  }
  if (i < 0 || i >= n) {
    in = false;
    return 0;
  }
  return i;
}

// out = A u = -L u, L the 12th-order Laplacian (weights w[0..6] already
// scaled by 1/h^2), FP64, and the workgroup's part of u . out.  A workgroup
// owns 64 x 8 points (two rows per lane) and marches along z: 13 planes of its
// points in a register queue renamed by phase, the current plane and its halo
// double-buffered in LDS.  HBM-bound (16 B a point): one thread per point with
// 37 cached reads took 323 us on 255^3, 0.82 TB/s of those bytes, plus 56 us
// for the separate product; this form 101 us with it.
struct W12 {
  double w[R12 + 1];
};
constexpr int kLTX = 64, kLTY = 8, kLW = kLTX + 2 * R12, kLRows = kLTY + 2 * R12;
__global__ __launch_bounds__(256) void lap12_kernel(const double* __restrict__ u, double* __restrict__ out, Grid g,
                                                    W12 w, March m, double* __restrict__ part) {
  __shared__ double buf[2][kLRows * kLW];
  __shared__ double red[4];
  const Tile t = march_tile(m, g.nz);
  const int tid = threadIdx.x, lx = tid & 63, ly = tid >> 6;
  const int x0 = t.bx * kLTX, y0 = t.by * kLTY;
  const int pp = g.nx * g.ny;
  int off[2];
  bool own[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int x = x0 + lx, y = y0 + ly + 4 * i;
    own[i] = x < g.nx && y < g.ny;
    off[i] = own[i] ? x + g.nx * y : 0;
  }
  // halo cells of this lane: 3 of the 12 y-halo rows, and one of the 12 x-halo
  // columns for the first 96 lanes.  A cell inside the tile's rows but past
  // the grid (ragged tiles) lies in the points' own range and is loaded as a
  // halo is (wrapped, or zero).
  int hoff[4], hl[4];
  bool hin[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int x, y, l;
    bool in = true;
    if (j < 3) {
      const int r = ly + 4 * j;  // 0..11
      x = x0 + lx;
      y = r < R12 ? y0 - R12 + r : y0 + kLTY + (r - R12);
      l = (r < R12 ? r : kLTY + r) * kLW + R12 + lx;
    } else {
      const int r = tid / (2 * R12), c = tid % (2 * R12);
      in = r < kLTY;
      x = c < R12 ? x0 - R12 + c : x0 + kLTX + (c - R12);
      y = y0 + r;
      l = in ? (R12 + r) * kLW + (c < R12 ? c : kLTX + c) : 0;
    }
    hl[j] = (j == 3 && !in) ? -1 : l;
    x = axis(x, g.nx, g.periodic, in);
    y = axis(y, g.ny, g.periodic, in);
    hin[j] = in;
    hoff[j] = in ? x + g.nx * y : 0;
  }
  // own cells past a ragged edge hold the wrapped neighbour (periodic) or zero
  int coff[2];
  bool cin[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    bool in = true;
    const int x = axis(x0 + lx, g.nx, g.periodic, in), y = axis(y0 + ly + 4 * i, g.ny, g.periodic, in);
    cin[i] = in;
    coff[i] = in ? x + g.nx * y : 0;
  }
  auto plane = [&](int z, bool& in) { return static_cast<int64_t>(axis(z, g.nz, g.periodic, in)) * pp; };
  auto ldc = [&](int i, int z) {
    bool in = cin[i];
    const int64_t zo = plane(z, in);
    const double v = u[zo + coff[i]];
    return in ? v : 0.0;
  };
  auto ldh = [&](int j, int z) {
    bool in = hin[j];
    const int64_t zo = plane(z, in);
    const double v = u[zo + hoff[j]];
    return in ? v : 0.0;
  };
  double q[2][Q12], fr[2], hv[4];
#pragma unroll
  for (int s = 0; s < Q12; ++s)
#pragma unroll
    for (int i = 0; i < 2; ++i) q[i][s] = ldc(i, t.z0 - R12 + s);
#pragma unroll
  for (int i = 0; i < 2; ++i) fr[i] = ldc(i, t.z0 + 1 + R12);
#pragma unroll
  for (int j = 0; j < 4; ++j) hv[j] = ldh(j, t.z0);
  double acc = 0.0;
  auto step = [&](auto phc, int z) {
    constexpr int PH = decltype(phc)::value;
    auto QS = [](int s2) { return (s2 + PH) % Q12; };
    double* b = buf[z & 1];
#pragma unroll
    for (int i = 0; i < 2; ++i) b[(R12 + ly + 4 * i) * kLW + R12 + lx] = q[i][QS(R12)];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (hl[j] >= 0) b[hl[j]] = hv[j];
#pragma unroll
    for (int j = 0; j < 4; ++j) hv[j] = ldh(j, z + 1);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double* c = b + (R12 + ly + 4 * i) * kLW + R12 + lx;
      const double ctr = q[i][QS(R12)];
      double s = 3.0 * w.w[0] * ctr;
#pragma unroll
      for (int p = 1; p <= R12; ++p)
        s += w.w[p] * ((c[p] + c[-p]) + (c[p * kLW] + c[-p * kLW]) + (q[i][QS(R12 + p)] + q[i][QS(R12 - p)]));
      if (own[i]) {
        out[static_cast<int64_t>(z) * pp + off[i]] = -s;
        acc -= ctr * s;
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      q[i][QS(0)] = fr[i];
      fr[i] = ldc(i, z + 2 + R12);
    }
  };
  using std::integral_constant;
  for (int z = t.z0; z < t.z1; z += Q12) {
    step(integral_constant<int, 0>{}, z);
    if (z + 1 < t.z1) step(integral_constant<int, 1>{}, z + 1); else break;
    if (z + 2 < t.z1) step(integral_constant<int, 2>{}, z + 2); else break;
    if (z + 3 < t.z1) step(integral_constant<int, 3>{}, z + 3); else break;
    if (z + 4 < t.z1) step(integral_constant<int, 4>{}, z + 4); else break;
    if (z + 5 < t.z1) step(integral_constant<int, 5>{}, z + 5); else break;
    if (z + 6 < t.z1) step(integral_constant<int, 6>{}, z + 6); else break;
    if (z + 7 < t.z1) step(integral_constant<int, 7>{}, z + 7); else break;
    if (z + 8 < t.z1) step(integral_constant<int, 8>{}, z + 8); else break;
    if (z + 9 < t.z1) step(integral_constant<int, 9>{}, z + 9); else break;
    if (z + 10 < t.z1) step(integral_constant<int, 10>{}, z + 10); else break;
    if (z + 11 < t.z1) step(integral_constant<int, 11>{}, z + 11); else break;
    if (z + 12 < t.z1) step(integral_constant<int, 12>{}, z + 12); else break;
  }
  const double tot = block_total(acc, red);
  if (tid == 0) part[blockIdx.x] = tot;
}

// Constant stencil of a level: centre, face, edge and corner weights (the
// Galerkin operators of the 7-point Laplacian keep its symmetry; the finest
// level has no edge and corner terms), and the damped Jacobi factor omega / c0.
struct SLev {
  float c0, c1, c2, c3, s;
};

// 1-D coarse neighbours of fine index i: two (index, weight) pairs, the
// second's weight zero when the fine point lies on a coarse one.
struct Pair1 {
  int a, b;
  float wa, wb;
};
__device__ __forceinline__ Pair1 coarse_pair(int i, int m, int periodic) {
  Pair1 r;
  if (periodic) {
    r.a = i >> 1;
    r.b = (i & 1) ? (r.a + 1 == m ? 0 : r.a + 1) : r.a;
    r.wa = (i & 1) ? 0.5f : 1.0f;
    r.wb = (i & 1) ? 0.5f : 0.0f;
  } else if (i & 1) {
    r.a = r.b = i >> 1;
    r.wa = 1.0f;
    r.wb = 0.0f;
  } else {
    const int k = i >> 1;
    r.a = max(k - 1, 0);
    r.b = min(k, m - 1);
    r.wa = k >= 1 ? 0.5f : 0.0f;
    r.wb = k < m ? 0.5f : 0.0f;
  }
  return r;
}
// (P_x P_y xc) of coarse plane K at fine (i, j); zero planes beyond a face
__device__ __forceinline__ float sheet(const float* __restrict__ xc, const Grid& gc, const Pair1& px, const Pair1& py,
                                       int K) {
  if (gc.periodic)
    K = K == gc.nz ? 0 : K;
  else if (K < 0 || K >= gc.nz)
    return 0.0f;
  const float* p = xc + static_cast<int64_t>(gc.nx) * gc.ny * K;
  const float* r = p + gc.nx * py.a;
  float v = py.wa * (px.wa * r[px.a] + px.wb * r[px.b]);
  if (py.wb != 0.0f) {  // uniform along a row
    const float* r2 = p + gc.nx * py.b;
    v += py.wb * (px.wa * r2[px.a] + px.wb * r2[px.b]);
  }
  return v;
}

// Marching V-cycle kernels.  A workgroup owns a 64 x TY tile (TY / 4 rows per
// lane) and a z range; each plane of the smoothed field (value() at the tile
// and a one-cell ring) is staged in LDS once and reduced there to its centre,
// face and corner sums, and the sums of three consecutive planes give A x.
// Every field is read once per launch from HBM; what a launch moves is the
// comment at its kind.  On 255^3 the five finest-level stages of a V-cycle
// take 235 us (8 sweep, residual, transfer and conversion launches of 40 to
// 100 us each before: one thread per point, a cached read per stencil entry).
//   kFirst : two damped Jacobi sweeps from zero: x = s r + s (r - A s r)  (read r, write x)
//   kJac   : one sweep x' = x + s (r - A x)                             (read x, r, write x')
//   kProlJac: the same from x + P xc                                    (read x, r, xc / 8, write x')
//   kLast  : kJac of the finest level with r read in FP64, and the parts of
//            r . x', sum x' and sum r
//   kRestr : t = r - A x, and its restriction P^T t                     (read x, r, write rc / 8)
enum MarchKind { kFirst, kJac, kProlJac, kLast, kRestr };
struct MArgs {
  const float* x;
  const float* r;
  const double* r64;
  const float* xc;
  float* out;
  Grid g, gc;
  SLev c;
  March m;
  double* part;   // kLast: three planes of gridDim.x values
};
constexpr int kVX = 64, kVW = kVX + 2;
template <int KIND>
struct MarchTile {
  static constexpr int TY = KIND == kRestr ? 16 : 8;
  static constexpr int P = TY / 4;
  static constexpr int RING = 2 * kVW + 2 * TY;  // ring cells, at most one per lane
};
template <int KIND, bool SEVEN>
__global__ __launch_bounds__(256) void march_kernel(MArgs A) {
  constexpr int TY = MarchTile<KIND>::TY, P = MarchTile<KIND>::P, RING = MarchTile<KIND>::RING;
  static_assert(RING <= 256, "one ring cell per lane");
  __shared__ float buf[2][(TY + 2) * kVW];
  __shared__ float tb[KIND == kRestr ? 2 : 1][KIND == kRestr ? TY * kVX : 1];
  __shared__ double red[3][4];
  const Grid g = A.g;
  const int nplanes = KIND == kRestr ? A.gc.nz : g.nz;  // coarse planes are dealt out when restricting
  const Tile t = march_tile(A.m, nplanes);
  const int tid = threadIdx.x, lx = tid & 63, ly = tid >> 6;
  // restricting tiles overlap by two cells: every coarse point's 27 fine
  // neighbours lie in one tile; fine coordinate fo + 2 I + {0, 1, 2}
  const int fo = g.periodic ? -1 : 0;
  const int x0 = KIND == kRestr ? t.bx * (kVX - 2) + fo : t.bx * kVX;
  const int y0 = KIND == kRestr ? t.by * (TY - 2) + fo : t.by * TY;
  const int z0 = KIND == kRestr ? 2 * t.z0 + fo : t.z0;
  const int z1 = KIND == kRestr ? 2 * t.z1 + fo + 1 : t.z1;
  const int64_t pp = static_cast<int64_t>(g.nx) * g.ny;
  int cx = 0, cy[P], coff[P];
  bool cin[P], own[P];
#pragma unroll
  for (int i = 0; i < P; ++i) {
    bool in = true;
    const int y = y0 + ly + 4 * i;
    cx = axis(x0 + lx, g.nx, g.periodic, in);
    cy[i] = axis(y, g.ny, g.periodic, in);
    cin[i] = in;
    own[i] = x0 + lx >= 0 && x0 + lx < g.nx && y >= 0 && y < g.ny;
    coff[i] = cx + g.nx * cy[i];
  }
  // this lane's ring cell
  int hx = 0, hy = 0, hl = -1;
  bool hin = false;
  if (tid < RING) {
    int rx, ry;
    if (tid < 2 * kVW) {
      rx = tid % kVW - 1;
      ry = tid < kVW ? -1 : TY;
    } else {
      const int e = tid - 2 * kVW;
      rx = (e & 1) ? kVX : -1;
      ry = e >> 1;
    }
    hl = (ry + 1) * kVW + rx + 1;
    hin = true;
    hx = axis(x0 + rx, g.nx, g.periodic, hin);
    hy = axis(y0 + ry, g.ny, g.periodic, hin);
  }
  const float* __restrict__ src = KIND == kFirst ? A.r : A.x;
  // smoothed field, zero beyond a face.  Called for consecutive planes of a
  // cell: with the prolongation added, sh keeps the cell's last coarse sheet,
  // so a new one is formed every second plane only.
  auto value = [&](int x, int y, int z, bool in, const Pair1& px, const Pair1& py, float& sh, bool start) -> float {
    const bool in_xy = in;
    const int zz = axis(z, g.nz, g.periodic, in);
    float v = in ? src[x + static_cast<int64_t>(g.nx) * y + pp * zz] : 0.0f;
    if constexpr (KIND == kProlJac) {
      if (!in_xy) return 0.0f;
      // fine plane on a coarse one (k = z / 2) or between k - 1 and k
      // (zero faces, even z) or k and k + 1 (periodic, odd z)
      const bool between = g.periodic ? (zz & 1) != 0 : (z & 1) == 0;
      const int kb = g.periodic ? (zz + 1) >> 1 : z >> 1;
      if (start) sh = sheet(A.xc, A.gc, px, py, between ? kb - 1 : kb);
      if (between) {
        const float nw = sheet(A.xc, A.gc, px, py, kb);
        v += in ? 0.5f * (sh + nw) : 0.0f;
        sh = nw;
      } else {
        v += in ? sh : 0.0f;
      }
    }
    return v;
  };
  Pair1 px{}, py[P], hpx{}, hpy{};
  float sh[P], hsh = 0.0f;
  if constexpr (KIND == kProlJac) {
    px = coarse_pair(cx, A.gc.nx, g.periodic);
    hpx = coarse_pair(hx, A.gc.nx, g.periodic);
    hpy = coarse_pair(hy, A.gc.ny, g.periodic);
#pragma unroll
    for (int i = 0; i < P; ++i) py[i] = coarse_pair(cy[i], A.gc.ny, g.periodic);
  }
  auto rhs = [&](int i, int z) -> float {
    bool in = cin[i];
    const int zz = axis(z, g.nz, g.periodic, in);
    if (KIND == kFirst || KIND == kLast || !in) return 0.0f;
    return A.r[coff[i] + pp * zz];
  };
  float vn[P], hn;  // the plane staged next
#pragma unroll
  for (int i = 0; i < P; ++i) vn[i] = value(cx, cy[i], z0 - 1, cin[i], px, py[i], sh[i], true);
  hn = value(hx, hy, z0 - 1, hin, hpx, hpy, hsh, true);
  float c[3][P], f[3][P], d[3][P];  // centre, face sum, corner sum of the last three planes
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int q = 0; q < 3; ++q) c[q][i] = f[q][i] = d[q][i] = 0.0f;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  float racc = 0.0f;  // restriction: running sum of this lane's coarse point
  for (int s = z0 - 1; s <= z1; ++s) {
    float* b = buf[s & 1];
#pragma unroll
    for (int i = 0; i < P; ++i) b[(1 + ly + 4 * i) * kVW + 1 + lx] = vn[i];
    if (hl >= 0) b[hl] = hn;
    float rz[P];
    double r64[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      c[0][i] = c[1][i];
      f[0][i] = f[1][i];
      d[0][i] = d[1][i];
      c[1][i] = c[2][i];
      f[1][i] = f[2][i];
      d[1][i] = d[2][i];
      c[2][i] = vn[i];
      rz[i] = rhs(i, s - 1);
      if constexpr (KIND == kLast) r64[i] = (own[i] && s - 1 >= z0) ? A.r64[coff[i] + pp * (s - 1)] : 0.0;
    }
    if (s < z1) {
#pragma unroll
      for (int i = 0; i < P; ++i) vn[i] = value(cx, cy[i], s + 1, cin[i], px, py[i], sh[i], false);
      hn = value(hx, hy, s + 1, hin, hpx, hpy, hsh, false);
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const float* q = b + (1 + ly + 4 * i) * kVW + 1 + lx;
      f[2][i] = (q[-1] + q[1]) + (q[-kVW] + q[kVW]);
      if constexpr (!SEVEN) d[2][i] = (q[-kVW - 1] + q[-kVW + 1]) + (q[kVW - 1] + q[kVW + 1]);
    }
    const int z = s - 1;  // plane whose three neighbours are now known
    if (z < z0) continue;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      float ax = A.c.c0 * c[1][i] + A.c.c1 * (f[1][i] + (c[0][i] + c[2][i]));
      if constexpr (!SEVEN)
        ax += A.c.c2 * (d[1][i] + (f[0][i] + f[2][i])) + A.c.c3 * (d[0][i] + d[2][i]);
      if constexpr (KIND == kRestr) {
        // points beyond a Dirichlet face hold no residual
        bool in = cin[i];
        (void)axis(z, g.nz, g.periodic, in);
        tb[z & 1][(ly + 4 * i) * kVX + lx] = in ? rz[i] - ax : 0.0f;
      } else if (own[i]) {
        const int64_t p = coff[i] + pp * z;
        if constexpr (KIND == kFirst) {
          const float x1 = A.c.s * c[1][i];
          A.out[p] = x1 + A.c.s * (c[1][i] - A.c.s * ax);
        } else if constexpr (KIND == kLast) {
          const float zn = c[1][i] + A.c.s * (static_cast<float>(r64[i]) - ax);
          A.out[p] = zn;
          a0 += r64[i] * static_cast<double>(zn);
          a1 += static_cast<double>(zn);
          a2 += r64[i];
        } else {
          A.out[p] = c[1][i] + A.c.s * (rz[i] - ax);
        }
      }
    }
    if constexpr (KIND == kRestr) {
      lds_barrier();
      constexpr int CX = kVX / 2 - 1, CY = TY / 2 - 1;  // coarse points of a tile
      const int I = tid % CX, J = tid / CX;
      if (J < CY) {
        const float* q = tb[z & 1] + (2 * J) * kVX + 2 * I;
        const float s2 = 0.25f * ((q[0] + q[2]) + (q[2 * kVX] + q[2 * kVX + 2])) +
                         0.5f * ((q[1] + q[2 * kVX + 1]) + (q[kVX] + q[kVX + 2])) + q[kVX + 1];
        const int rel = z - z0;  // 0, 1, 2 of the first coarse plane, then 2, 3, 4 of the next, ...
        if (rel & 1) {
          racc += s2;
        } else {
          racc += 0.5f * s2;
          const int K = t.z0 + rel / 2 - 1, gi = t.bx * CX + I, gj = t.by * CY + J;
          if (rel > 0 && gi < A.gc.nx && gj < A.gc.ny)
            A.out[gi + static_cast<int64_t>(A.gc.nx) * (gj + static_cast<int64_t>(A.gc.ny) * K)] = racc;
          racc = 0.5f * s2;
        }
      }
    }
  }
  if constexpr (KIND == kLast) {
    const double t0 = block_total(a0, red[0]), t1 = block_total(a1, red[1]), t2 = block_total(a2, red[2]);
    if (tid == 0) {
      A.part[blockIdx.x] = t0;
      A.part[gridDim.x + blockIdx.x] = t1;
      A.part[2 * gridDim.x + blockIdx.x] = t2;
    }
  }
}

// The coarse end of the V-cycle (levels of at most kTailPts points) in one
// workgroup, fields in LDS: barriers in place of launches.  Right-hand side
// of its first level in rc, solution out in xc.  Zero-Dirichlet fields carry a
// ring of zeros, so no neighbour is tested; a point's coordinates are decoded
// once, into LDS.  The arguments live in device memory: a level-indexed
// argument block is copied to scratch by the compiler.
constexpr int kTailPts = 8192, kTailLevels = 8, kTailThreads = 1024;
struct TailLevel {
  int nx, ny, nz, n;
  int sx, sy;          // LDS strides of y and z (in cells)
  int x, w, r, at;     // LDS offsets: solution, work, right-hand side (n values), packed coordinates (n)
  SLev c;
};
struct TailArgs {
  int nl, lds;         // levels, LDS words
  TailLevel lev[kTailLevels];
};
// cells of a level's x and w fields (with their ring when zero-Dirichlet)
inline int tail_cells(const Grid& g) {
  return g.periodic ? g.nx * g.ny * g.nz : (g.nx + 2) * (g.ny + 2) * (g.nz + 2);
}
template <int PER>
__global__ __launch_bounds__(kTailThreads) void tail_kernel(const TailArgs* __restrict__ A,
                                                            const float* __restrict__ rc, float* __restrict__ xc) {
  extern __shared__ float lds[];
  const int tid = threadIdx.x;
  const int nl = A->nl;
  for (int q = tid; q < A->lds; q += kTailThreads) lds[q] = 0.0f;
  __syncthreads();
  for (int l = 0; l < nl; ++l) {
    const TailLevel v = A->lev[l];
    int* at = reinterpret_cast<int*>(lds) + v.at;
    for (int p = tid; p < v.n; p += kTailThreads) {
      const int i = p % v.nx, jk = p / v.nx;
      at[p] = i | (jk % v.ny) << 10 | (jk / v.ny) << 20;
    }
  }
  {
    float* r = lds + A->lev[0].r;
    for (int p = tid; p < A->lev[0].n; p += kTailThreads) r[p] = rc[p];
  }
  __syncthreads();
  // cell of a point in x and w
  auto cell = [](const TailLevel& v, int i, int j, int k) {
    return PER ? i + j * v.sx + k * v.sy : (i + 1) + (j + 1) * v.sx + (k + 1) * v.sy;
  };
  auto apply = [&](const float* f, const TailLevel& v, int i, int j, int k) {
    int ox[3], oy[3], oz[3];
    if (PER) {
      ox[0] = i == 0 ? v.nx - 1 : i - 1;
      ox[1] = i;
      ox[2] = i + 1 == v.nx ? 0 : i + 1;
      oy[0] = (j == 0 ? v.ny - 1 : j - 1) * v.sx;
      oy[1] = j * v.sx;
      oy[2] = (j + 1 == v.ny ? 0 : j + 1) * v.sx;
      oz[0] = (k == 0 ? v.nz - 1 : k - 1) * v.sy;
      oz[1] = k * v.sy;
      oz[2] = (k + 1 == v.nz ? 0 : k + 1) * v.sy;
    } else {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        ox[d] = i + d;
        oy[d] = (j + d) * v.sx;
        oz[d] = (k + d) * v.sy;
      }
    }
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c3 = 0; c3 < 3; ++c3)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const float* row = f + (oy[b] + oz[c3]);
#pragma unroll
        for (int a = 0; a < 3; ++a) s[(a != 1) + (b != 1) + (c3 != 1)] += row[ox[a]];
      }
    return v.c.c0 * s[0] + v.c.c1 * s[1] + v.c.c2 * s[2] + v.c.c3 * s[3];
  };
  auto each = [&](const TailLevel& v, auto&& fn) {
    const int* at = reinterpret_cast<const int*>(lds) + v.at;
    for (int p = tid; p < v.n; p += kTailThreads) {
      const int q = at[p];
      fn(p, q & 1023, (q >> 10) & 1023, q >> 20);
    }
    __syncthreads();
  };
  auto sweeps = [&](const TailLevel& v, int n) {  // n (even) Jacobi sweeps of x
    float *x = lds + v.x, *w = lds + v.w;
    const float* r = lds + v.r;
    for (int q = 0; q < n; ++q) {
      each(v, [&](int p, int i, int j, int k) {
        const int o = cell(v, i, j, k);
        w[o] = x[o] + v.c.s * (r[p] - apply(x, v, i, j, k));
      });
      float* t = x;
      x = w;
      w = t;
    }
  };
  auto zero_sweeps = [&](const TailLevel& v, int n) {  // n (even) sweeps from zero
    float *x = lds + v.x, *w = lds + v.w;
    const float* r = lds + v.r;
    each(v, [&](int p, int i, int j, int k) { w[cell(v, i, j, k)] = v.c.s * r[p]; });
    each(v, [&](int p, int i, int j, int k) {
      const int o = cell(v, i, j, k);
      x[o] = w[o] + v.c.s * (r[p] - apply(w, v, i, j, k));
    });
    sweeps(v, n - 2);
  };
  for (int l = 0; l + 1 < nl; ++l) {
    const TailLevel v = A->lev[l], vc = A->lev[l + 1];
    zero_sweeps(v, kNu);
    const float *x = lds + v.x, *r = lds + v.r;
    float *w = lds + v.w, *rn = lds + vc.r;
    each(v, [&](int p, int i, int j, int k) { w[cell(v, i, j, k)] = r[p] - apply(x, v, i, j, k); });
    each(vc, [&](int p, int I, int J, int K) {  // P^T: fine(I) + {-1, 0, 1}, weights 1/2, 1, 1/2 per axis
      int ox[3], oy[3], oz[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (PER) {
          ox[d] = 2 * I + d - 1 < 0 ? v.nx - 1 : 2 * I + d - 1;  // nx is even: the upper end never wraps
          oy[d] = (2 * J + d - 1 < 0 ? v.ny - 1 : 2 * J + d - 1) * v.sx;
          oz[d] = (2 * K + d - 1 < 0 ? v.nz - 1 : 2 * K + d - 1) * v.sy;
        } else {
          ox[d] = 2 * I + d + 1;
          oy[d] = (2 * J + d + 1) * v.sx;
          oz[d] = (2 * K + d + 1) * v.sy;
        }
      }
      float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c3 = 0; c3 < 3; ++c3)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
          for (int a = 0; a < 3; ++a) s[(a != 1) + (b != 1) + (c3 != 1)] += w[ox[a] + oy[b] + oz[c3]];
      rn[p] = s[0] + 0.5f * s[1] + 0.25f * s[2] + 0.125f * s[3];
    });
  }
  zero_sweeps(A->lev[nl - 1], kNuCoarse);
  for (int l = nl - 2; l >= 0; --l) {
    const TailLevel v = A->lev[l], vc = A->lev[l + 1];
    float* x = lds + v.x;
    const float* e = lds + vc.x;
    each(v, [&](int, int i, int j, int k) {  // x += P e, the two coarse neighbours of each axis
      int ox[2], oy[2], oz[2];
      if (PER) {  // even: the coincident coarse point twice, halved
        ox[0] = i >> 1;
        ox[1] = (i & 1) ? (ox[0] + 1 == vc.nx ? 0 : ox[0] + 1) : ox[0];
        const int b0 = j >> 1, b1 = (j & 1) ? (b0 + 1 == vc.ny ? 0 : b0 + 1) : b0;
        const int c0 = k >> 1, c1 = (k & 1) ? (c0 + 1 == vc.nz ? 0 : c0 + 1) : c0;
        oy[0] = b0 * vc.sx;
        oy[1] = b1 * vc.sx;
        oz[0] = c0 * vc.sy;
        oz[1] = c1 * vc.sy;
      } else {  // ring cells of the coarse field are zero
        ox[0] = (i + 1) >> 1;
        ox[1] = (i >> 1) + 1;
        oy[0] = ((j + 1) >> 1) * vc.sx;
        oy[1] = ((j >> 1) + 1) * vc.sx;
        oz[0] = ((k + 1) >> 1) * vc.sy;
        oz[1] = ((k >> 1) + 1) * vc.sy;
      }
      float s = 0.0f;
#pragma unroll
      for (int c3 = 0; c3 < 2; ++c3)
#pragma unroll
        for (int b = 0; b < 2; ++b) s += e[ox[0] + oy[b] + oz[c3]] + e[ox[1] + oy[b] + oz[c3]];
      x[cell(v, i, j, k)] += 0.125f * s;
    });
    sweeps(v, kNu);
  }
  const TailLevel v = A->lev[0];
  const float* x = lds + v.x;
  each(v, [&](int p, int i, int j, int k) { xc[p] = x[cell(v, i, j, k)]; });
}

// ---- FP64 vectors of CG ------------------------------------------------------
// Device scalars: what one kernel leaves for the next.
enum Scal { kRz, kAlpha, kBeta, kMean, kScalars };
constexpr int kVecBlocks = 8192;  // workgroups of the vector kernels at most (255^3: 2,048 3 to 9 % slower, 512 75 %)

// fn(p) for every p < n: workgroups stride over chunks of 1,024 values, four
// a lane with their loads in flight together.
template <typename F>
__device__ __forceinline__ void each_value(int64_t n, F&& fn) {
  for (int64_t c = static_cast<int64_t>(blockIdx.x) * 1024; c < n; c += static_cast<int64_t>(gridDim.x) * 1024) {
    if (c + 1024 <= n) {
#pragma unroll
      for (int k = 0; k < 4; ++k) fn(c + threadIdx.x + 256 * k);
    } else {
      for (int64_t p = c + threadIdx.x; p < n; p += 256) fn(p);
    }
  }
}
// 0 f + 4 pi f: a non-finite f stays NaN as the sum a x + b y gave it
__device__ __forceinline__ double four_pi(double f) { return 0.0 * f + 4.0 * M_PI * f; }
__global__ __launch_bounds__(256) void charge_sum_kernel(const double* __restrict__ f, int64_t n,
                                                         double* __restrict__ part) {
  __shared__ double red[4];
  double s = 0.0;
  each_value(n, [&](int64_t p) { s += four_pi(f[p]); });
  const double t = block_total(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}
// r = 4 pi f (minus its mean when periodic), r in FP32, part of r . r
__global__ __launch_bounds__(256) void start_kernel(const double* __restrict__ f, int64_t n,
                                                    const double* __restrict__ sc, int periodic,
                                                    double* __restrict__ r, float* __restrict__ r32,
                                                    double* __restrict__ part) {
  __shared__ double red[4];
  const double mean = periodic ? sc[kMean] : 0.0;
  double s = 0.0;
  each_value(n, [&](int64_t p) {
    const double v = four_pi(f[p]) - mean;
    r[p] = v;
    r32[p] = static_cast<float>(v);
    s += v * v;
  });
  const double t = block_total(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}
// x += alpha p (last iteration's), p = z - mean + beta p; first: x = 0, p = z - mean
template <typename ZT>
__global__ __launch_bounds__(256) void direction_kernel(const ZT* __restrict__ z, int64_t n,
                                                        const double* __restrict__ sc, int first,
                                                        double* __restrict__ p, double* __restrict__ x) {
  const double alpha = sc[kAlpha], beta = sc[kBeta], mean = sc[kMean];
  each_value(n, [&](int64_t q) {
    const double zv = static_cast<double>(z[q]) - mean;
    if (first) {
      x[q] = 0.0;
      p[q] = zv;
    } else {
      const double pv = p[q];
      x[q] += alpha * pv;
      p[q] = zv + beta * pv;
    }
  });
}
// r -= alpha Ap, r in FP32, part of r . r
__global__ __launch_bounds__(256) void update_kernel(const double* __restrict__ Ap, int64_t n,
                                                     const double* __restrict__ sc, double* __restrict__ r,
                                                     float* __restrict__ r32, double* __restrict__ part) {
  __shared__ double red[4];
  const double alpha = sc[kAlpha];
  double s = 0.0;
  each_value(n, [&](int64_t p) {
    const double v = r[p] - alpha * Ap[p];
    r[p] = v;
    r32[p] = static_cast<float>(v);
    s += v * v;
  });
  const double t = block_total(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}
// phi = x + alpha p, part of its sum
__global__ __launch_bounds__(256) void solution_kernel(const double* __restrict__ x, const double* __restrict__ p,
                                                       int64_t n, const double* __restrict__ sc,
                                                       double* __restrict__ phi, double* __restrict__ part) {
  __shared__ double red[4];
  const double alpha = sc[kAlpha];
  double s = 0.0;
  each_value(n, [&](int64_t q) {
    const double v = x[q] + alpha * p[q];
    phi[q] = v;
    s += v;
  });
  const double t = block_total(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}
__global__ __launch_bounds__(256) void shift_kernel(double* __restrict__ y, int64_t n, const double* __restrict__ sc) {
  const double mean = sc[kMean];
  each_value(n, [&](int64_t p) { y[p] -= mean; });
}
__global__ __launch_bounds__(256) void zero_kernel(double* __restrict__ y, int64_t n) {
  each_value(n, [&](int64_t p) { y[p] = 0.0; });
}
__global__ void to_f32_kernel(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
  const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p < n) b[p] = static_cast<float>(a[p]);
}
__global__ void to_f64_kernel(const float* __restrict__ a, double* __restrict__ b, int64_t n) {
  const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p < n) b[p] = static_cast<double>(a[p]);
}

// Sums np partials (per plane, fixed order) in one workgroup and leaves the
// scalar that follows from them:
//   kFinMean  : mean = sum / n
//   kFinAlpha : alpha = rz / sum                     (sum = p . A p)
//   kFinNorm  : *host = sum                          (r . r, pinned host memory)
//   kFinBeta  : rz' = r.z - mean(z) sum(r), beta = rz' / rz, mean = mean(z)
//               (planes r.z, sum z, sum r; the means only when periodic)
enum FinKind { kFinMean, kFinAlpha, kFinNorm, kFinBeta };
__global__ __launch_bounds__(1024) void finish_kernel(const double* __restrict__ part, int np, int kind, int periodic,
                                                      int first, double n, double* __restrict__ sc,
                                                      double* __restrict__ host) {
  __shared__ double red[3][16];
  const int planes = (kind == kFinBeta && periodic) ? 3 : 1;
  for (int q = 0; q < planes; ++q) {
    double s = 0.0;
    for (int b = threadIdx.x; b < np; b += 1024) s += part[static_cast<int64_t>(q) * np + b];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = s;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double t[3] = {0.0, 0.0, 0.0};
  for (int q = 0; q < planes; ++q)
    for (int w = 0; w < 16; ++w) t[q] += red[q][w];
  if (kind == kFinMean) {
    sc[kMean] = t[0] / n;
  } else if (kind == kFinAlpha) {
    sc[kAlpha] = sc[kRz] / t[0];
  } else if (kind == kFinNorm) {
    *host = t[0];
    __threadfence_system();
  } else {
    const double mean = periodic ? t[1] / n : 0.0;
    const double rz = t[0] - mean * t[2];
    sc[kBeta] = first ? 0.0 : rz / sc[kRz];
    sc[kRz] = rz;
    sc[kMean] = mean;
  }
}

void check(const char* what) { XLS_LAUNCH_CHECK(what); }

int coarse_size(int m, bool periodic) {
  if (periodic) return (m % 2 == 0 && m / 2 >= 4) ? m / 2 : -1;
  return (m % 2 == 1 && (m - 1) / 2 >= 3) ? (m - 1) / 2 : -1;
}

// Galerkin stencil P^T A P of a constant 27-point stencil a with trilinear P:
// c(J) = sum_{u, v} p(u) a(v) p(u + v - 2 J), offsets in {-1, 0, 1}^3.
std::array<double, 27> galerkin(const std::array<double, 27>& a) {
  auto p1 = [](int d) { return d == 0 ? 1.0 : (d == -1 || d == 1 ? 0.5 : 0.0); };
  std::array<double, 27> c{};
  for (int J = 0; J < 27; ++J) {
    const int jx = J % 3 - 1, jy = (J / 3) % 3 - 1, jz = J / 9 - 1;
    double s = 0.0;
    for (int U = 0; U < 27; ++U) {
      const int ux = U % 3 - 1, uy = (U / 3) % 3 - 1, uz = U / 9 - 1;
      for (int V = 0; V < 27; ++V) {
        if (a[V] == 0.0) continue;
        const int vx = V % 3 - 1, vy = (V / 3) % 3 - 1, vz = V / 9 - 1;
        const int wx = ux + vx - 2 * jx, wy = uy + vy - 2 * jy, wz = uz + vz - 2 * jz;
        const double pu = p1(ux) * p1(uy) * p1(uz), pwv = p1(wx) * p1(wy) * p1(wz);
        s += pu * a[V] * pwv;
      }
    }
    c[J] = s;
  }
  return c;
}

}  // namespace

struct xls_poisson_s {
  Grid g{};
  double h = 0.0;
  int64_t nd = 0;
  std::vector<Grid> lev;
  std::vector<SLev> st;
  int tail = 0;                      // first level of the one-workgroup end (lev.size() when there is none)
  TailArgs* tail_args = nullptr;
  size_t tail_lds = 0;
  std::vector<float*> xl, rl, tl;  // per level: solution, right-hand side, work
  double *b = nullptr, *x = nullptr, *r = nullptr, *p = nullptr, *Ap = nullptr, *part = nullptr, *sc = nullptr;
  double* norm = nullptr;            // pinned host value of the last kFinNorm
  hipEvent_t ev = nullptr;
  hipStream_t s = nullptr;
  W12 w12{};
  ~xls_poisson_s() {
    if (s) (void)hipStreamSynchronize(s);
    for (auto* q : xl) dfree(q);
    for (auto* q : rl) dfree(q);
    for (auto* q : tl) dfree(q);
    void* ps[] = {b, x, r, p, Ap, part, sc, tail_args};
    for (void* q : ps) dfree(q);
    if (norm) (void)hipHostFree(norm);
    if (ev) (void)hipEventDestroy(ev);
    if (s) (void)hipStreamDestroy(s);
  }
  int64_t size(int l) const { return static_cast<int64_t>(lev[l].nx) * lev[l].ny * lev[l].nz; }
};

namespace {

// z ranges of a marching launch: about `wgs` workgroups, of at least min_tz
// planes each (a range re-reads 2 planes of a V-cycle field and 12 of the
// Laplacian's).  On 255^3, us per launch at 512 / 768 / 1,024 / 1,536 / 2,048
// workgroups: Laplacian 109 / 101 / 104 / - / 110, finest-level sweeps 98 / - /
// 70 / 62 / 66, restriction 85 / - / 65 / 58 / 66.
constexpr int kLapWgs = 768, kLevelWgs = 1536;
March march_of(int nx, int ny, int nz, int tx, int ty, int min_tz, int wgs, unsigned& blocks) {
  March m;
  m.nbx = (nx + tx - 1) / tx;
  m.nby = (ny + ty - 1) / ty;
  const int64_t xy = static_cast<int64_t>(m.nbx) * m.nby;
  const int64_t nzt = std::max<int64_t>(1, std::min<int64_t>(wgs / xy, nz / min_tz));
  m.tz = static_cast<int>((nz + nzt - 1) / nzt);
  const int64_t nb = xy * ((nz + m.tz - 1) / m.tz);
  if (nb > 0x7fffffff) fail(XLS_ERR_INVALID_ARG, "grid too large");
  blocks = static_cast<unsigned>(nb);
  return m;
}
March lap_march(const Grid& g, unsigned& blocks) {
  return march_of(g.nx, g.ny, g.nz, kLTX, kLTY, 2, kLapWgs, blocks);
}
template <int KIND>
March level_march(const Grid& g, const Grid& gc, unsigned& blocks) {
  constexpr int TY = MarchTile<KIND>::TY;
  if (KIND == kRestr) return march_of(gc.nx, gc.ny, gc.nz, kVX / 2 - 1, TY / 2 - 1, 2, kLevelWgs, blocks);
  return march_of(g.nx, g.ny, g.nz, kVX, TY, 4, kLevelWgs, blocks);
}
unsigned vec_blocks(int64_t n) { return static_cast<unsigned>(std::min<int64_t>(kVecBlocks, (n + 1023) / 1024)); }

void finish(xls_poisson_s* P, unsigned np, FinKind kind, int periodic, int first) {
  hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(1024), 0, P->s, P->part, static_cast<int>(np),
                     static_cast<int>(kind), periodic, first, static_cast<double>(P->nd), P->sc, P->norm);
  check("finish_kernel");
}

template <int KIND>
unsigned march(xls_poisson_s* P, int l, const float* x, float* out) {
  MArgs A{};
  A.x = x;
  A.r = P->rl[l];
  A.r64 = P->r;
  A.out = out;
  A.g = P->lev[l];
  A.c = P->st[l];
  A.part = P->part;
  if (KIND == kProlJac || KIND == kRestr) {
    A.gc = P->lev[l + 1];
    A.xc = P->xl[l + 1];
  }
  unsigned nb = 0;
  A.m = level_march<KIND>(A.g, A.gc, nb);
  if (l == 0)
    hipLaunchKernelGGL((march_kernel<KIND, true>), dim3(nb), dim3(256), 0, P->s, A);
  else if constexpr (KIND != kLast)  // the finest level's only
    hipLaunchKernelGGL((march_kernel<KIND, false>), dim3(nb), dim3(256), 0, P->s, A);
  else
    fail(XLS_ERR_INVALID_ARG, "the last sweep is the finest level's");
  check("march_kernel");
  return nb;
}

// x_l = (V-cycle from level l) r_l; with dots (level 0) the last sweep also
// leaves the parts of r . z, sum z and sum r.  Returns its workgroups.
unsigned vcycle(xls_poisson_s* P, int l, bool dots) {
  const int L = static_cast<int>(P->lev.size());
  if (l >= P->tail) {
    if (P->g.periodic)
      hipLaunchKernelGGL(tail_kernel<1>, dim3(1), dim3(kTailThreads), P->tail_lds, P->s, P->tail_args, P->rl[l],
                         P->xl[l]);
    else
      hipLaunchKernelGGL(tail_kernel<0>, dim3(1), dim3(kTailThreads), P->tail_lds, P->s, P->tail_args, P->rl[l],
                         P->xl[l]);
    check("tail_kernel");
    return 0;
  }
  float *x = P->xl[l], *t = P->tl[l];
  march<kFirst>(P, l, nullptr, x);
  if (l == L - 1) {
    static_assert(kNuCoarse % 2 == 0, "sweeps end in x");
    for (int k = 2; k < kNuCoarse; ++k) {
      if (k == kNuCoarse - 1 && dots) return march<kLast>(P, l, x, t);
      march<kJac>(P, l, x, t);
      std::swap(x, t);
    }
    return 0;
  }
  static_assert(kNu == 2, "pre- and post-smoothing are fused for two sweeps");
  march<kRestr>(P, l, x, P->rl[l + 1]);
  vcycle(P, l + 1, false);
  march<kProlJac>(P, l, x, t);
  if (dots) return march<kLast>(P, l, t, x);
  march<kJac>(P, l, t, x);
  return 0;
}

}  // namespace

extern "C" {

int xls_poisson_create(const int32_t* n, double h, int32_t bc, int32_t max_levels, xls_poisson_t* out) {
  return guarded([&]() -> int {
    if (!out || !n) fail(XLS_ERR_INVALID_ARG, "NULL argument");
    for (int a = 0; a < 3; ++a)
      if (n[a] < 1) fail(XLS_ERR_INVALID_ARG, "grid size must be >= 1");
    if (!(h > 0) || !std::isfinite(h)) fail(XLS_ERR_INVALID_ARG, "h must be finite and > 0");
    if (bc != XLS_BC_PERIODIC && bc != XLS_BC_DIRICHLET0) fail(XLS_ERR_INVALID_ARG, "unknown bc");
    if (max_levels < 0 || max_levels > 16) fail(XLS_ERR_INVALID_ARG, "max_levels must be in [0, 16]");
    const int64_t nd = static_cast<int64_t>(n[0]) * n[1] * n[2];
    if (nd >= (int64_t(1) << 31)) fail(XLS_ERR_INVALID_ARG, "grid too large");
    auto* P = new xls_poisson_s();
    try {
      P->g = Grid{n[0], n[1], n[2], bc == XLS_BC_PERIODIC ? 1 : 0};
      P->h = h;
      P->nd = nd;
      XLS_HIP(hipStreamCreateWithFlags(&P->s, hipStreamNonBlocking));
      // 12th-order weights scaled by 1/h^2
      double f[2 * R12 + 1];
      f[0] = 1.0;
      for (int i = 1; i <= 2 * R12; ++i) f[i] = f[i - 1] * i;
      double sw = 0.0;
      for (int q = 1; q <= R12; ++q) {
        P->w12.w[q] = 2.0 * ((q % 2 == 1) ? 1.0 : -1.0) * f[R12] * f[R12] /
                      (static_cast<double>(q) * q * f[R12 - q] * f[R12 + q]) / (h * h);
        sw += P->w12.w[q];
      }
      P->w12.w[0] = -2.0 * sw;
      // levels and their constant stencils
      std::array<double, 27> a{};
      a[13] = 6.0 / (h * h);
      a[12] = a[14] = a[10] = a[16] = a[4] = a[22] = -1.0 / (h * h);
      const int maxl = max_levels > 0 ? max_levels : 8;
      P->lev.push_back(P->g);
      for (;;) {
        // centre, face, edge and corner entries of the (symmetric) stencil
        SLev s{static_cast<float>(a[13]), static_cast<float>(a[12]), static_cast<float>(a[9]),
               static_cast<float>(a[0]), 0.0f};
        s.s = kOmega / s.c0;
        P->st.push_back(s);
        if (static_cast<int>(P->lev.size()) >= maxl) break;
        const Grid& g = P->lev.back();
        const int cx = coarse_size(g.nx, g.periodic), cy = coarse_size(g.ny, g.periodic),
                  cz = coarse_size(g.nz, g.periodic);
        if (cx < 0 || cy < 0 || cz < 0) break;
        P->lev.push_back(Grid{cx, cy, cz, g.periodic});
        a = galerkin(a);
      }
      for (size_t l = 0; l < P->lev.size(); ++l) {
        const size_t m = static_cast<size_t>(P->size(static_cast<int>(l)));
        P->xl.push_back(dalloc<float>(m));
        P->rl.push_back(dalloc<float>(m));
        P->tl.push_back(dalloc<float>(m));
      }
      double** vs[] = {&P->b, &P->x, &P->r, &P->p, &P->Ap};
      for (double** v : vs) *v = dalloc<double>(nd);
      // the levels small enough for one workgroup's LDS (never the finest:
      // its last sweep forms the dot products)
      P->tail = 1;
      const int L = static_cast<int>(P->lev.size());
      while (P->tail < L && P->size(P->tail) > kTailPts) ++P->tail;
      if (L - P->tail > kTailLevels) P->tail = L;
      if (P->tail < L) {
        TailArgs T{};
        T.nl = L - P->tail;
        for (int q = 0; q < T.nl; ++q) {
          const Grid& g = P->lev[P->tail + q];
          TailLevel& v = T.lev[q];
          const int pad = g.periodic ? 0 : 2, cells = tail_cells(g);
          v.nx = g.nx;
          v.ny = g.ny;
          v.nz = g.nz;
          v.n = g.nx * g.ny * g.nz;
          v.sx = g.nx + pad;
          v.sy = v.sx * (g.ny + pad);
          v.x = T.lds;
          v.w = v.x + cells;
          v.r = v.w + cells;
          v.at = v.r + v.n;
          v.c = P->st[P->tail + q];
          T.lds = v.at + v.n;
        }
        P->tail_lds = 4 * static_cast<size_t>(T.lds);
        if (P->tail_lds > 160 * 1024) {  // flat levels whose ring outweighs their points
          P->tail = L;
        } else {
          P->tail_args = dalloc<TailArgs>(1);
          XLS_HIP(hipMemcpyAsync(P->tail_args, &T, sizeof(T), hipMemcpyHostToDevice, P->s));
          XLS_HIP(hipStreamSynchronize(P->s));
          ensure_dyn_smem(P->g.periodic ? reinterpret_cast<const void*>(tail_kernel<1>)
                                        : reinterpret_cast<const void*>(tail_kernel<0>), P->tail_lds);
        }
      }
      unsigned nlap = 0, nlast = 0;
      (void)lap_march(P->g, nlap);
      (void)level_march<kLast>(P->g, P->g, nlast);
      P->part = dalloc<double>(std::max<size_t>({kVecBlocks, nlap, 3 * static_cast<size_t>(nlast)}));
      P->sc = dalloc<double>(kScalars);
      XLS_HIP(hipHostMalloc(reinterpret_cast<void**>(&P->norm), sizeof(double), hipHostMallocDefault));
      XLS_HIP(hipEventCreateWithFlags(&P->ev, hipEventDisableTiming));
    } catch (...) {
      delete P;
      throw;
    }
    *out = P;
    return XLS_OK;
  });
}

void xls_poisson_destroy(xls_poisson_t P) { delete P; }

int xls_poisson_vcycle(xls_poisson_t P, const double* r, double* z) {
  return guarded([&]() -> int {
    if (!P || !r || !z) fail(XLS_ERR_INVALID_ARG, "NULL argument");
    if (!finite_all(r, P->nd)) fail(XLS_ERR_INVALID_ARG, "r not finite");
    XLS_HIP(hipMemcpyAsync(P->r, r, P->nd * 8, hipMemcpyHostToDevice, P->s));
    hipLaunchKernelGGL(to_f32_kernel, dim3(nblk(P->nd, 256)), dim3(256), 0, P->s, P->r, P->rl[0], P->nd);
    vcycle(P, 0, false);
    hipLaunchKernelGGL(to_f64_kernel, dim3(nblk(P->nd, 256)), dim3(256), 0, P->s, P->xl[0], P->Ap, P->nd);
    check("xls_poisson_vcycle");
    XLS_HIP(hipMemcpyAsync(z, P->Ap, P->nd * 8, hipMemcpyDeviceToHost, P->s));
    XLS_HIP(hipStreamSynchronize(P->s));
    return XLS_OK;
  });
}

}  // extern "C"

namespace {

// CG on the handle's device vectors from f into phi (either may be a caller's
// device array).  One iteration is two vector kernels, the Laplacian and the
// V-cycle, with alpha and beta formed on the device; the host reads r . r
// once per iteration, while the GPU is already in the next V-cycle (unless the
// last ratio of norms says that this iteration is the last: then that V-cycle
// would be wasted).  To 1e-10: 255^3 26.1 -> 10.7 ms, periodic 64 x 96 x 48
// 6.2 -> 2.05 ms (six vector passes, three dot products with a host wait each
// and 74 launches an iteration before; 24 now).
void solve_on_device(xls_poisson_t P, const double* f, double* phi, double tol, int32_t max_iter, int32_t precond,
                     double* info, std::chrono::steady_clock::time_point t0) {
  const int64_t nd = P->nd;
  const int per = P->g.periodic;
  const unsigned nv = vec_blocks(nd);
  const dim3 gv(nv), bl(256);
  if (per) {
    hipLaunchKernelGGL(charge_sum_kernel, gv, bl, 0, P->s, f, nd, P->part);
    finish(P, nv, kFinMean, per, 0);
  }
  hipLaunchKernelGGL(start_kernel, gv, bl, 0, P->s, f, nd, P->sc, per, P->r, P->rl[0], P->part);
  check("start_kernel");
  auto read_norm = [&]() {
    XLS_HIP(hipEventSynchronize(P->ev));
    return std::sqrt(*P->norm);
  };
  auto send_norm = [&]() {
    finish(P, nv, kFinNorm, 0, 0);
    XLS_HIP(hipEventRecord(P->ev, P->s));
  };
  // z = B r and the scalars of the next direction
  auto precondition = [&](int first) {
    if (precond)
      finish(P, vcycle(P, 0, true), kFinBeta, per, first);
    else
      finish(P, nv, kFinBeta, 0, first);  // z = r: the parts of r . r
  };
  send_norm();
  const double nb = read_norm();
  int it = 0;
  double rel = 0.0;
  if (nb > 0.0) {
    const float* z32 = P->xl[0];
    precondition(1);
    rel = 1.0;
    double ratio = 1.0;
    for (it = 1; it <= max_iter; ++it) {
      if (precond)
        hipLaunchKernelGGL(direction_kernel<float>, gv, bl, 0, P->s, z32, nd, P->sc, it == 1, P->p, P->x);
      else
        hipLaunchKernelGGL(direction_kernel<double>, gv, bl, 0, P->s, P->r, nd, P->sc, it == 1, P->p, P->x);
      unsigned nl = 0;
      const March m = lap_march(P->g, nl);
      hipLaunchKernelGGL(lap12_kernel, dim3(nl), bl, 0, P->s, P->p, P->Ap, P->g, P->w12, m, P->part);
      check("lap12_kernel");
      finish(P, nl, kFinAlpha, 0, 0);
      hipLaunchKernelGGL(update_kernel, gv, bl, 0, P->s, P->Ap, nd, P->sc, P->r, P->rl[0], P->part);
      check("update_kernel");
      send_norm();
      const bool ahead = it < max_iter && rel * ratio > 2.0 * tol;
      if (ahead) precondition(0);
      const double prev = rel;
      rel = read_norm() / nb;
      ratio = rel / prev;
      if (!(rel > tol)) break;  // NaN ends the loop too
      if (!ahead && it < max_iter) precondition(0);
    }
    if (it > max_iter) it = max_iter;
    hipLaunchKernelGGL(solution_kernel, gv, bl, 0, P->s, P->x, P->p, nd, P->sc, phi, P->part);
    check("solution_kernel");
    if (per) {
      finish(P, nv, kFinMean, per, 0);
      hipLaunchKernelGGL(shift_kernel, gv, bl, 0, P->s, phi, nd, P->sc);
      check("shift_kernel");
    }
  } else {
    hipLaunchKernelGGL(zero_kernel, gv, bl, 0, P->s, phi, nd);
    check("zero_kernel");
  }
  XLS_HIP(hipStreamSynchronize(P->s));
  if (info) {
    info[0] = it;
    info[1] = rel;
    info[2] = static_cast<double>(P->lev.size());
    info[3] = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  }
}

void check_solve_args(xls_poisson_t P, const void* f, const void* phi, double tol, int32_t max_iter) {
  if (!P || !f || !phi) fail(XLS_ERR_INVALID_ARG, "NULL argument");
  if (!(tol > 0) || max_iter < 1) fail(XLS_ERR_INVALID_ARG, "tol must be > 0 and max_iter >= 1");
}

}  // namespace

extern "C" {

int xls_poisson_solve(xls_poisson_t P, const double* f, double* phi, double tol, int32_t max_iter,
                      int32_t precond, double* info) {
  return guarded([&]() -> int {
    check_solve_args(P, f, phi, tol, max_iter);
    if (!finite_all(f, P->nd)) fail(XLS_ERR_INVALID_ARG, "f not finite");
    const auto t0 = std::chrono::steady_clock::now();
    XLS_HIP(hipMemcpyAsync(P->b, f, P->nd * 8, hipMemcpyHostToDevice, P->s));
    solve_on_device(P, P->b, P->b, tol, max_iter, precond, info, t0);
    XLS_HIP(hipMemcpyAsync(phi, P->b, P->nd * 8, hipMemcpyDeviceToHost, P->s));
    XLS_HIP(hipStreamSynchronize(P->s));
    if (info) info[3] = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return XLS_OK;
  });
}

int xls_poisson_solve_device(xls_poisson_t P, const double* f, double* phi, double tol, int32_t max_iter,
                             int32_t precond, double* info) {
  return guarded([&]() -> int {
    check_solve_args(P, f, phi, tol, max_iter);
    check_device_range(f, P->nd * 8);
    check_device_range(phi, P->nd * 8);
    const auto t0 = std::chrono::steady_clock::now();
    solve_on_device(P, f, phi, tol, max_iter, precond, info, t0);
    return XLS_OK;
  });
}

}  // extern "C"
