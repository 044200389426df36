// Full-dimension SOV estimate of log Phi_D(x / scale) (Genz's method over all D
// variables), the comparator the paper checks the Vecchia approximation
// against (Section 3.1, Figures 1-4), on the plan's ordering and covariance.
//
//   1. full_cov_build: the dense D x D covariance (plan order, FP64) and b = x / scale;
//   2. blocked right-looking Cholesky, one launch per 32 columns (chol_step):
//      the panel's factor, its rows and the update of the trailing lower
//      triangle on the FP64 matrix cores; the factor goes to the upper triangle
//      as L^T, so that a column of L is contiguous;
//   3. full_sov: one workgroup per 16 to 144 lattice points for the whole chain:
//      products by the earlier dimensions' y on the FP64 matrix cores
//      (v_mfma_f64_16x16x4), the recursion of 16 dimensions at a time with a
//      point per lane; it leaves {max, sum exp(. - max)} of each 16 points' log products;
//   4. full_final (one workgroup, fixed-order trees): per shift l_r = log mean
//      over points, then log F = log mean_r exp(l_r) and the delta-method SE
//      over the shifts.
// Lattice: Z_j from the first D - 1 primes; the shift of dimension j in
// replicate r is SplitMix64 output 2^63 + r 2^32 + j of the call's seed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "device_cov.h"
#include "device_math_f64.h"
#include "lattice.h"
#include "qmc_f64.h"
#include "runtime.h"
#include "vecchia.h"

namespace vecchia {
namespace {

constexpr int kCholB = 32;     // Cholesky block
constexpr int kFsWavePts = 16; // lattice points per wave (one MFMA column tile)
constexpr int kFsTile = 16;    // dimensions per tile (one MFMA row tile)
constexpr int kFsWaves = 8;    // waves per workgroup: row tiles per block of dimensions
constexpr int kFsBufs = 4;        // product steps in flight, less one

// v_mfma_f64_16x16x4f64, D = A B + C with A 16 x 4, B 4 x 16: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16], and holds D[4 e + l / 16][l % 16] in
// element e of its four-double result (checked on gfx950).
typedef double fs_d4 __attribute__((ext_vector_type(4)));

struct CovArgs {
  const double* xs;
  const double* ys;
  const double* covmat;
  const int32_t* perm;
  const double* x;
  double inv_scale, sigma2, range, nugget, nu;
  int32_t family;
};

__global__ __launch_bounds__(256) void full_cov_build(CovArgs a, int64_t D, double* __restrict__ A,
                                                      double* __restrict__ b) {
  const int64_t j = (int64_t)blockIdx.x * 16 + (threadIdx.x & 15);
  const int64_t i = (int64_t)blockIdx.y * 16 + (threadIdx.x >> 4);
  if (i >= D || j > i) return;
  double v;
  if (a.covmat) {
    v = a.covmat[i * D + j];
  } else {
#pragma clang fp contract(off)
    const double dx = a.xs[i] - a.xs[j];
    const double dy = a.ys[i] - a.ys[j];
    v = cov_kernel(sqrt(dx * dx + dy * dy), a.family, a.nu, a.sigma2, a.range);
    if (i == j) v += a.nugget;
  }
  A[i * D + j] = v;
  if (j == 0) b[i] = a.x[a.perm[i]] * a.inv_scale;
}

__device__ __forceinline__ double lane_value(double v, int lane) {   // lane uniform
  const uint64_t b = bits_of(v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return of_bits(((uint64_t)hi << 32) | lo);
}

// One step of the blocked right-looking Cholesky of the lower triangle, a launch
// per panel of kCholB columns: workgroup (tj, ti), tj <= ti, of 64 x 64 tiles of
// the trailing matrix [k0 + n, D).
//   1. Wave 0 factors the panel's diagonal block (lane r holds row r in
//      registers; a column's pivot and entries are read across lanes as scalar
//      operands) while the other waves stage the panel rows of the tile's rows
//      and columns in LDS.
//   2. One thread per staged row solves x L_kk^T = a (the pivots' reciprocals
//      from step 1, updates of the row's later entries independent of each other).
//   3. The tile is updated, A[i][j] -= sum_c x_i[c] x_j[c], each wave a 32 x 32
//      quarter as 2 x 2 tiles of v_mfma_f64_16x16x4.
// Every workgroup repeats steps 1 and 2 for its own tile: both are latency, and
// repeating them costs less than the two launches that would share them (and a
// factor written in place would be read by workgroups that have not started).
// The factor goes to the upper triangle as L^T, its diagonal's reciprocal to
// dinv; the lower triangle is left with the panels as they were before their
// own step. A non-positive pivot gives NaN from its column on. Bounded by the
// chain of launches: 26 us each at 2,500 dimensions, 79 of them, against 50 us
// for the three launches (factor, rows, update) of a panel before. (The factor's
// rows by LDS broadcasts instead of lane reads: 31 us, its registers spill.)
// Rows are multiplied by the pivots' reciprocals where a division would round once:
// over 16 instances of 400 to 1,000 dimensions log F is off from 25-digit values by
// 4.0e-15 (exponential) and 1.6e-15 (Matern with a nugget) relative on average, the
// three launches before, which divided, by 4.0e-15 and 2.7e-15.
__global__ __launch_bounds__(256) void chol_step(double* __restrict__ A, double* __restrict__ dinv, int64_t D,
                                                 int64_t k0, int n) {
  const int64_t base = k0 + n;
  const int64_t ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  __shared__ double P[128][kCholB + 1];          // panel rows: 0..63 the tile's rows, 64..127 its columns
  __shared__ double Lc[kCholB][kCholB];          // L_kk by columns: Lc[c][r]
  __shared__ double inv[kCholB];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wi = wv >> 1, wj = wv & 1;
  const int m = lane & 15, kq = lane >> 4;
  const int64_t i0 = base + ti * 64, c0 = base + tj * 64;
  if (wv == 0) {
    double c[kCholB];
#pragma unroll
    for (int p = 0; p < kCholB; ++p) c[p] = (lane < n && p <= lane) ? A[(k0 + lane) * D + k0 + p] : 0.0;
#pragma unroll
    for (int j = 0; j < kCholB; ++j) {
      if (j < n) {
        const double d = lane_value(c[j], j);
        // 1 / sqrt(d) by two Newton steps, then sqrt(d) = d / sqrt(d) corrected
        double r = __builtin_amdgcn_rsq(d);
        r = __builtin_fma(r, __builtin_fma(-d * r, 0.5 * r, 0.5), r);
        r = __builtin_fma(r, __builtin_fma(-d * r, 0.5 * r, 0.5), r);
        double g = d * r;
        g = __builtin_fma(__builtin_fma(-g, g, d), 0.5 * r, g);
        if (!(d > 0.0)) r = g = __builtin_nan("");
        c[j] = lane == j ? g : c[j] * r;
        if (lane == j) inv[j] = r;
        if (lane >= j && lane < kCholB) Lc[j][lane] = c[j];
#pragma unroll
        for (int p = j + 1; p < kCholB; ++p) c[p] = __builtin_fma(-lane_value(c[j], p), c[j], c[p]);
      }
    }
    if (ti == 0) {
#pragma unroll
      for (int j = 0; j < kCholB; ++j)
        if (j < n && lane > j && lane < n) A[(k0 + j) * D + k0 + lane] = c[j];
      if (lane < n) dinv[k0 + lane] = inv[lane];
    }
  } else {
    // rows past the matrix as zeros: their products are never stored
    for (int idx = tid - 64; idx < 128 * kCholB; idx += 192) {
      const int r = idx / kCholB, c = idx - r * kCholB;
      const int64_t row = r < 64 ? i0 + r : c0 + r - 64;
      P[r][c] = row < D ? A[row * D + k0 + c] : 0.0;
    }
  }
  // the tile, while the factor is under way
  double tile[2][2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = i0 + 32 * wi + 16 * a + 4 * e + kq, j = c0 + 32 * wj + 16 * b + m;
        tile[a][b][e] = (i < D && j <= i) ? A[i * D + j] : 0.0;
      }
  if (base >= D) return;   // the last panel: nothing below it (uniform over the grid)
  __syncthreads();
  if (tid < (ti == tj ? 64 : 128)) {
    double x[kCholB];
#pragma unroll
    for (int c = 0; c < kCholB; ++c) x[c] = P[tid][c];
#pragma unroll
    for (int c = 0; c < kCholB; ++c) {
      x[c] *= inv[c];
#pragma unroll
      for (int d = c + 1; d < kCholB; ++d) x[d] = __builtin_fma(-Lc[c][d], x[c], x[d]);
    }
#pragma unroll
    for (int c = 0; c < kCholB; ++c) P[tid][c] = x[c];
  }
  __syncthreads();
  if (tj == 0) {
    for (int idx = tid; idx < 64 * kCholB; idx += 256) {
      const int c = idx >> 6, r = idx & 63;
      if (i0 + r < D) A[(k0 + c) * D + i0 + r] = P[r][c];
    }
  }
  const double (*Pj)[kCholB + 1] = ti == tj ? P : P + 64;
  fs_d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = fs_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < kCholB / 4; ++ks) {
    const int c = 4 * ks + kq;
    const double a0 = P[32 * wi + m][c], a1 = P[32 * wi + 16 + m][c];
    const double b0 = Pj[32 * wj + m][c], b1 = Pj[32 * wj + 16 + m][c];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  }
  // acc[a][b] element e (the MFMA's output layout): row 32 wi + 16 a + 4 e + kq,
  // column 32 wj + 16 b + m of the tile
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = i0 + 32 * wi + 16 * a + 4 * e + kq, j = c0 + 32 * wj + 16 * b + m;
        if (i < D && j <= i) A[i * D + j] = tile[a][b][e] - acc[a][b][e];
      }
}

// log Phi(t), t < -kPhiNodeMax (or NaN, which stays), with e = Phi(t): log e while e is above
// 1e-197; below, -t^2/2 + log((1 - 1/t^2 + 1*3/t^4 - ...) / (|t| sqrt(2 pi))), whose
// first term left out is 3e-16 at t = -30; -inf where t^2 overflows.
__device__ __forceinline__ double log_ncdf_low(double t, double e) {
  const double h = t * t, z = div64(1.0, h);
  double p = 1.0 - 13.0 * z;
#pragma unroll
  for (int k = 11; k >= 1; k -= 2) p = __builtin_fma(-k * z, p, 1.0);
  const bool far = !(t > -30.0);
  if (h == HUGE_VAL) return -HUGE_VAL;
  return log64(far ? div64(p, -2.50662827463100050242 * t) : e) - (far ? 0.5 * h : 0.0);
}

// The larger of the two; NaN if either is (a covariance that is not positive definite).
__device__ __forceinline__ double max_nan(double a, double b) { return a >= b || a != a ? a : b; }

// L: D x D with L^T strictly above the diagonal (what is on and below it is not
// read as L); dinv: reciprocals of L's diagonal; b: D limits; Z: D - 1 generators;
// Y: per workgroup, earlier step of four dimensions and tile of 16 points, 64 y
// (dimension 4 s + lane / 16 of point lane % 16); part: {max, sum exp} per tile of points.
struct SovArgs {
  const double* L;
  const double* dinv;
  const double* b;
  const uint64_t* Z;
  double* Y;
  double2* part;
  int64_t D, N;
  uint64_t seed;
  int64_t tiles, all_tiles;   // 16-point tiles per shift, and of all shifts
  int64_t y_steps;            // steps of four dimensions in a workgroup's Y
};

// A point's recursion over rows Q.. of a tile (left of them below D):
//     e = Phi(t_q), log prod += log Phi(t_q), y_q = Phi^-1(max(w_q e, DBL_MIN)),
//     T[q'] -= L[q][q'] y_q for q' > q (L scaled by its rows' pivots, as T is).
// ty: the point's column of the staged tile (its y replace its limits); w: of the coordinates.
struct SovPoint {
  double T[kFsTile];
  double prod;   // of the tile's e outside the rare branch: at least 1e-272
  double lp;
};
template <int Q, int PT>
__device__ __forceinline__ void sov_rows(SovPoint& s, double* ty, const double* w, const double (*L)[kFsTile], int left,
                                         const double* nodes) {
  if (Q >= left) return;
  const double t = s.T[Q];
  double e = phi_nodes(nodes, fmax(fmin(t, kPhiNodeMax), -kPhiNodeMax));
  double f = e;
  if (__builtin_expect(any_lane(!(t >= -kPhiNodeMax)), 0)) {
    if (!(t >= -kPhiNodeMax)) {
      e = phi64(t);
      s.lp += log_ncdf_low(t, e);
      f = 1.0;
    }
  }
  s.prod *= f;
  double u, uc, side;
  {
    // the product rounds before 1 - u, as the quantile's argument is u itself
#pragma clang fp contract(off)
    u = w[Q * PT] * e;
    uc = 1.0 - u;
    side = u - 0.5;
  }
  const double q = fmin(u, uc);
  double y = __builtin_copysign(ninv_nodes(nodes, q), side);
  if (__builtin_expect(any_lane(!(q >= kNinvNodeMin)), 0)) {
    if (!(q >= kNinvNodeMin)) y = ninv64(fmax(u, 2.2250738585072014e-308));
  }
  ty[Q * PT] = y;
  double row[kFsTile];
#pragma unroll
  for (int c = Q + 1; c < kFsTile; ++c) row[c] = L[Q][c];
#pragma unroll
  for (int c = Q + 1; c < kFsTile; ++c) {
    s.T[c] = __builtin_fma(-row[c], y, s.T[c]);
    // stays here: moved to the step that uses T[c], it would keep y and row alive
    __asm__ volatile("" : "+v"(s.T[c]));
  }
  if constexpr (Q + 1 < kFsTile) sov_rows<Q + 1, PT>(s, ty, w, L, left, nodes);
}

// A workgroup owns C tiles of 16 consecutive lattice points for the whole chain.
// Dimensions go in tiles of 16 rows, kFsWaves tiles to a block (the first block
// takes the remainder), one row tile of the block per wave:
//  * Earlier blocks: acc = L[the wave's rows, 0..j0) y for the C point tiles by
//    v_mfma_f64_16x16x4: the A operand is L[j + m][c0 + k] (row c0 + k of the
//    upper triangle, 16 consecutive doubles per k), the B operands the y of
//    step c0 / 4 (512 consecutive bytes per point tile, read by every wave); the
//    loads of the next kFsBufs - 1 steps are in flight.
//  * The block's tiles in turn: the tile's wave leaves its scaled limits
//    (b - acc) / L_cc in LDS, the first waves run the recursion with a point per
//    lane, and the waves of the later tiles take the new y into their acc, while
//    all threads stage the next tile's lattice coordinates and triangle of L.
// So the product's matrix work is spread evenly over the compute unit's SIMDs
// whatever the number of points, and the recursion's vector work is done once
// per point; it leaves the matrix cores idle for the latency of its serial
// chain, about 1,000 clocks a dimension. With a wave per 16 points for both
// (each factor evaluated by four lanes, three waves on some SIMDs and two on
// others), 2,500 dimensions and 3607 x 10 points took 7.8 ms. Measured against
// one wave per 16 points with fitted ratios and the recursion's triangle in
// LDS: that case 14.6 -> 6.1 ms (the product alone is 3.0 ms at the FP64 matrix
// peak), 500 x 4 points 8.6 -> 1.7 ms, 900 dimensions and 10^4 x 10 points
// 8.3 -> 3.1 ms, 5,000 dimensions and 2000 x 10 points 32.3 -> 14.5 ms.
template <int C>
__global__ __launch_bounds__(64 * kFsWaves) __attribute__((amdgpu_waves_per_eu(kFsWaves / 4))) void full_sov(SovArgs a) {
  constexpr int PT = 16 * C;
  constexpr int kThreads = 64 * kFsWaves;
  __shared__ __align__(16) double nodes[2 * kNormNodes];
  __shared__ double ty[2][kFsTile][PT];    // a tile's limits, then its y
  __shared__ double wt[kFsTile][PT];       // its lattice coordinates
  __shared__ __align__(16) double Lt[kFsTile][kFsTile];   // Lt[q][c] = L_{j+c,j+q} / L_{j+c,j+c}, c > q
  load_nodes(nodes);
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6);
  const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (wg * C >= a.all_tiles) return;
  const int m = lane & 15, kq = lane >> 4;
  const int64_t D = a.D;
  double* __restrict__ Yw = a.Y + wg * a.y_steps * (64 * C);
  const int64_t n_tiles = (D + kFsTile - 1) / kFsTile;
  int block = (int)(n_tiles % kFsWaves);
  if (block == 0) block = kFsWaves;

  // point p of the workgroup: its shift and 1-based index (past the shift's or
  // the last shift's points: some point, its results unused)
  auto point = [&](int p, int64_t* shift, bool* live) {
    int64_t tile = wg * C + (p >> 4);
    *live = tile < a.all_tiles;
    if (!*live) tile = a.all_tiles - 1;
    *shift = (uint32_t)tile / (uint32_t)a.tiles;
    const int64_t pn = (tile - *shift * a.tiles) * 16 + (p & 15);
    *live = *live && pn < a.N;
    return (uint64_t)(pn < a.N ? pn : a.N - 1) + 1;
  };
  // entry (q, c) = (tid / 16, tid % 16) of the triangle, the reads past D inside the workspace
  double lt = 0.0;
  auto load_triangle = [&](int64_t j) {
    if (tid < kFsTile * kFsTile) {
      const int64_t row = j + (tid >> 4);
      lt = a.L[(row < D ? row : D - 1) * D + j + (tid & 15)] * a.dinv[j + (tid & 15)];
    }
  };
  auto stage = [&](int64_t j) {
    if (tid < kFsTile * kFsTile) Lt[tid >> 4][tid & 15] = lt;
    for (int idx = tid; idx < kFsTile * PT; idx += kThreads) {
      const int q = idx / PT, p = idx - q * PT;
      int64_t r;
      bool live;
      const uint64_t pt = point(p, &r, &live);
      const int64_t dim = j + q;
      const uint64_t z = a.Z[dim < D - 1 ? dim : (D > 1 ? D - 2 : 0)];   // the last dimension's y is not used
      wt[q][p] = lattice_coord_f64(pt * z + splitmix64(a.seed, (1ULL << 63) | ((uint64_t)r << 32) | (uint64_t)dim));
    }
  };

  SovPoint s;
  s.lp = 0.0;
  int buf = 0;
  for (int64_t j0 = 0; j0 < D;) {
    fs_d4 acc[C];
#pragma unroll
    for (int i = 0; i < C; ++i) acc[i] = fs_d4{0.0, 0.0, 0.0, 0.0};
    const int64_t jw = j0 + (int64_t)wv * kFsTile;   // the wave's row tile
    const bool mine = wv < block;
    load_triangle(j0);
    const int steps = (int)(j0 / 4);   // a multiple of 4
    if (steps > 0) {   // then block == kFsWaves
      // columns past D in the last tile read other entries (of the next row,
      // which exists: c < j0); their sums are never used
      const double* __restrict__ aA = a.L + (int64_t)kq * D + jw + m;
      const double* __restrict__ aB = Yw + lane;
      double av[kFsBufs], bv[kFsBufs][C];
      auto load_step = [&](int st, int u) {
        av[u] = aA[(int64_t)st * 4 * D];
        const double* __restrict__ br = aB + (int64_t)st * (64 * C);
#pragma unroll
        for (int i = 0; i < C; ++i) bv[u][i] = br[64 * i];
      };
      // the loads past the last step re-read it: with every load unconditional
      // the compiler's wait counts stay exact across the loop
#pragma unroll
      for (int u = 0; u < kFsBufs - 1; ++u) load_step(u, u);
      for (int st = 0; st < steps; st += kFsBufs) {
#pragma unroll
        for (int u = 0; u < kFsBufs; ++u) {
          const int nx = st + u + kFsBufs - 1;
          load_step(nx < steps ? nx : steps - 1, (u + kFsBufs - 1) % kFsBufs);
#pragma unroll
          for (int i = 0; i < C; ++i)
            acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u][i], acc[i], 0, 0, 0);
        }
      }
    }
    // acc[i] element e (the MFMA's output layout): row 4 e + kq, point 16 i + m;
    // rows past D in the last tile take what follows b in the workspace, unused
    auto leave_limits = [&](int64_t j) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double bq = a.b[j + 4 * e + kq], dq = a.dinv[j + 4 * e + kq];
#pragma unroll
        for (int i = 0; i < C; ++i) ty[buf][4 * e + kq][16 * i + m] = (bq - acc[i][e]) * dq;
      }
    };
    const bool keep = j0 + (int64_t)block * kFsTile < D;   // a later block reads the y
    if (wv == 0) leave_limits(j0);
    stage(j0);
#pragma unroll 1
    for (int i = 0; i < block; ++i) {
      const int64_t j = j0 + (int64_t)i * kFsTile;
      const bool later = mine && wv > i;
      // A operands of the update after the recursion
      double nv[4] = {0.0, 0.0, 0.0, 0.0};
      if (later) {
#pragma unroll
        for (int st = 0; st < 4; ++st) nv[st] = a.L[(j + 4 * st + kq) * D + jw + m];
      }
      __syncthreads();
      const int left = (int)(D - j < kFsTile ? D - j : kFsTile);
      if (tid < PT) {
#pragma unroll
        for (int q = 0; q < kFsTile; ++q) s.T[q] = ty[buf][q][tid];
        s.prod = 1.0;
        sov_rows<0, PT>(s, &ty[buf][0][tid], &wt[0][tid], Lt, left, nodes);
        s.lp += log(s.prod);
      }
      __syncthreads();
      if (keep) {   // the whole tile is below D
        for (int idx = tid; idx < kFsTile * PT; idx += kThreads) {
          const int l = idx & 63, ct = (idx >> 6) % C, st = (idx >> 6) / C;
          Yw[((j / 4 + st) * C + ct) * 64 + l] = ty[buf][4 * st + (l >> 4)][16 * ct + (l & 15)];
        }
      }
      if (i + 1 < block) load_triangle(j + kFsTile);
      if (later) {
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
          for (int ct = 0; ct < C; ++ct)
            acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(nv[st], ty[buf][4 * st + kq][16 * ct + m], acc[ct], 0, 0, 0);
      }
      buf ^= 1;
      if (i + 1 < block) {
        if (wv == i + 1) leave_limits(j + kFsTile);
        stage(j + kFsTile);
      }
    }
    __syncthreads();   // the block's y are in Y before its readers, and ty is free
    j0 += (int64_t)block * kFsTile;
    block = kFsWaves;
  }
  // each point tile's {max, sum exp(lp - max)} over its live points (16 lanes)
  if (tid < PT) {
    int64_t r;
    bool live;
    point(tid, &r, &live);
    double mx = live ? s.lp : -HUGE_VAL;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) mx = max_nan(mx, __shfl_xor(mx, o, 16));
    double x = (live && mx > -HUGE_VAL) ? exp(s.lp - mx) : 0.0;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) x += __shfl_xor(x, o, 16);
    const int64_t tile = wg * C + (tid >> 4);
    if (m == 0 && tile < a.all_tiles) a.part[tile] = make_double2(mx, x);
  }
}

template <int C>
hipError_t launch_sov(const SovArgs& a, hipStream_t s) {
  const int64_t groups = (a.all_tiles + C - 1) / C;
  const unsigned gx = (unsigned)std::min<int64_t>(groups, 1 << 20), gy = (unsigned)((groups + gx - 1) / gx);
  hipLaunchKernelGGL(full_sov<C>, dim3(gx, gy), dim3(64 * kFsWaves), 0, s, a);
  return hipGetLastError();
}

// Point tiles per workgroup: of the compiled counts the one with the least
// rounds x (product + recursion) for one workgroup per compute unit, D / 8 clocks per
// dimension and point tile for the product on four SIMDs, 1,000 for the recursion.
int sov_tiles(int64_t all_tiles, int64_t D, int n_cu) {
  int best = 1;
  double least = 0.0;
  for (int c : {1, 2, 3, 4, 6, 9}) {
    const int64_t groups = (all_tiles + c - 1) / c;
    const double t = (double)((groups + n_cu - 1) / n_cu) * (c * (D / 8.0) + 1000.0);
    if (c == 1 || t < least) {
      best = c;
      least = t;
    }
  }
  return best;
}

// One workgroup of 256: per shift r, l_r = log mean over points from the waves'
// {max, sum exp} partials (strided partial reductions, then a fixed tree, so the
// result does not depend on scheduling); then log F = log mean_r exp(l_r) and
// the delta-method SE over shifts. A NaN partial makes both NaN.
__global__ __launch_bounds__(256) void full_final(const double2* __restrict__ part, int nblk, int R, int64_t N,
                                                  double* __restrict__ out) {
  __shared__ double red[256];
  const int tid = threadIdx.x;
  auto tree = [&](double v, bool is_max) {
    red[tid] = v;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (tid < o) red[tid] = is_max ? max_nan(red[tid], red[tid + o]) : red[tid] + red[tid + o];
      __syncthreads();
    }
    const double res = red[0];
    __syncthreads();
    return res;
  };
  auto logmean = [&](int r) {
    const double2* __restrict__ pr = part + (int64_t)r * nblk;
    double mx = -HUGE_VAL;
    for (int k = tid; k < nblk; k += 256) mx = max_nan(mx, pr[k].x);
    const double M = tree(mx, true);
    if (!(M > -HUGE_VAL)) return M;
    double sm = 0.0;
    for (int k = tid; k < nblk; k += 256) {
      const double2 v = pr[k];
      if (v.x > -HUGE_VAL) sm += v.y * exp(v.x - M);
    }
    return M + log(tree(sm, false)) - log((double)N);
  };
  double top = -HUGE_VAL;
  for (int r = 0; r < R; ++r) top = max_nan(top, logmean(r));
  double logF = top, se = __builtin_nan("");
  if (top > -HUGE_VAL) {
    double sum = 0.0;
    for (int r = 0; r < R; ++r) sum += exp(logmean(r) - top);
    logF = top + log(sum) - log((double)R);
    if (R > 1) {
      double acc = 0.0;
      for (int r = 0; r < R; ++r) {
        const double d = exp(logmean(r) - logF) - 1.0;
        acc += d * d;
      }
      se = sqrt(acc / ((double)R * (R - 1)));
    }
  }
  if (tid == 0) {
    out[0] = logF;
    out[1] = se;
  }
}

}  // namespace
}  // namespace vecchia

extern "C" vecchia_status vecchia_full_logcdf(vecchia_plan_t plan, const double* x_dev, double scale,
                                              const vecchia_cov* cov_override, const vecchia_qmc* q,
                                              double* out_dev, void* hip_stream) {
  using namespace vecchia;
  if (!plan || !q || !x_dev || !out_dev) return set_error(VECCHIA_E_INVALID, "null pointer");
  std::string why;
  if (!valid_qmc(*q, &why)) return set_error(VECCHIA_E_INVALID, why);
  if (q->precision != VECCHIA_FP64) return set_error(VECCHIA_E_INVALID, "the full-dimension estimator runs in FP64");
  if (q->n_shifts > 1024) return set_error(VECCHIA_E_INVALID, "n_shifts must be at most 1024 here");
  if (plan->n_obs > 0) return set_error(VECCHIA_E_INVALID, "not defined for a censored plan");
  if (!(std::isfinite(scale) && scale > 0)) return set_error(VECCHIA_E_INVALID, "scale must be finite and > 0");
  const vecchia_cov c = cov_override ? *cov_override : plan->cov;
  if (cov_override) {
    if (!valid_cov(c, &why)) return set_error(VECCHIA_E_INVALID, why);
    if (!plan->matrix && (c.family != plan->cov.family || (c.family == VECCHIA_COV_MATERN && c.nu != plan->cov.nu)))
      return set_error(VECCHIA_E_INVALID, "covariance override must keep the plan's family and nu");
  }
  const int64_t D = plan->D, N = q->n_points, R = q->n_shifts;
  const int64_t S = N * R;   // points
  // the limit: A (D x D), b (D), (D - 1) y for each of the S points and the partials
  // (what is allocated below pads a shift's points to 16: at most 15 R D doubles more, 4.9 GB)
  const int64_t n_head = D * D + D + std::max<int64_t>(1, D - 1) * S;
  const int64_t n_head_even = n_head + (n_head & 1);
  const double bytes = 8.0 * (double)n_head_even + 16.0 * R * ((N + kFsWavePts - 1) / kFsWavePts + 3);
  if (D > 40000 || bytes > 64e9)
    return set_error(VECCHIA_E_INVALID, "the full-dimension estimator needs D <= 40000 and at most 64 GB of workspace");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  std::lock_guard<std::mutex> lk(plan->mu);
  hipError_t e = hipSuccess;
  int dev = 0;
  e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_error(e, "device query");
  const uint64_t* Zt = device_lattice_table_n(dev, (int)std::max<int64_t>(1, D - 1), &e);
  if (!Zt) return hip_error(e, "lattice table");
  // workspace: A, b, dinv (D each), the y of all blocks but the last (64 per
  // step of four dimensions and point tile, whole workgroups), the partials at
  // a 16-byte offset; the slack covers reads past b and dinv in a last, partial tile
  hipDeviceProp_t prop{};
  int n_cu = 256;
  if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0) n_cu = prop.multiProcessorCount;
  const int64_t tiles = (N + kFsWavePts - 1) / kFsWavePts, all_tiles = tiles * R;
  const int per_group = sov_tiles(all_tiles, D, n_cu);
  const int64_t held_tiles = (all_tiles + per_group - 1) / per_group * per_group;
  const int64_t y_steps = std::max<int64_t>(0, (D + kFsTile - 1) / kFsTile - kFsWaves) * (kFsTile / 4);
  const int64_t n_y = D * D + 2 * D, n_part = (n_y + (n_y & 1)) + 64 * y_steps * held_tiles;
  const size_t need = (size_t)(8 * n_part + 16 * all_tiles) + 1024;
  if (plan->full_bytes < need) {
    hipFree(plan->d_full);
    plan->d_full = nullptr;
    plan->full_bytes = 0;
    e = hipMalloc(&plan->d_full, need);
    if (e != hipSuccess) {
      plan->d_full = nullptr;
      return hip_error(e, "full-dimension workspace");
    }
    plan->full_bytes = need;
  }
  double* A = reinterpret_cast<double*>(plan->d_full);
  double* b = A + D * D;
  double* dinv = b + D;
  double* Y = A + n_y + (n_y & 1);
  double2* part = reinterpret_cast<double2*>(A + n_part);
  CovArgs ca{plan->d_xs, plan->d_ys, plan->d_cov, plan->d_perm, x_dev, 1.0 / scale, c.sigma2, c.range, c.nugget,
             c.family == VECCHIA_COV_EXPONENTIAL ? 0.5 : c.nu, c.family};
  const unsigned t16 = (unsigned)((D + 15) / 16);
  hipLaunchKernelGGL(full_cov_build, dim3(t16, t16), dim3(256), 0, s, ca, D, A, b);
  e = hipGetLastError();
  for (int64_t k0 = 0; k0 < D && e == hipSuccess; k0 += kCholB) {
    const int n = (int)std::min<int64_t>(kCholB, D - k0);
    const int64_t rest = D - k0 - n;
    const unsigned t = (unsigned)std::max<int64_t>(1, (rest + 63) / 64);   // 64 x 64 tiles of the trailing triangle
    hipLaunchKernelGGL(chol_step, dim3(t, t), dim3(256), 0, s, A, dinv, D, k0, n);
    e = hipGetLastError();
  }
  // measurement hook: HIP events around the product-and-recursion kernel,
  // recorded with its D(D-1)/2 FMAs per point
  hipEvent_t pa = nullptr, pb = nullptr;
  const bool prof = e == hipSuccess && profiling_enabled() && profile_events(&pa, &pb) == hipSuccess;
  if (prof) e = hipEventRecord(pa, s);
  if (e == hipSuccess) {
    const SovArgs sa{A, dinv, b, Zt, Y, part, D, N, q->seed, tiles, all_tiles, y_steps};
    switch (per_group) {
      case 1: e = launch_sov<1>(sa, s); break;
      case 2: e = launch_sov<2>(sa, s); break;
      case 3: e = launch_sov<3>(sa, s); break;
      case 4: e = launch_sov<4>(sa, s); break;
      case 6: e = launch_sov<6>(sa, s); break;
      default: e = launch_sov<9>(sa, s); break;
    }
  }
  if (prof && e == hipSuccess) {
    e = hipEventRecord(pb, s);
    if (e == hipSuccess) profile_record(VECCHIA_PROFILE_FULL_SOV, VECCHIA_FP64, pa, pb, D * (D - 1) / 2 * N * R);
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(full_final, dim3(1), dim3(256), 0, s, part, (int)tiles, (int)R, N, out_dev);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return hip_error(e, "full-dimension launch");
  return VECCHIA_OK;
}
