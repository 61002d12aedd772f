// Kernel ridge regression in float64: the linear system of Sec. 2 (the one
// the paper's preconditioned conjugate gradients solve iteratively), solved
// here directly by Cholesky factorisation, which is its exact solution.
//
//   lambda = ridge_rel mean(diag K_train),  A = K_train + lambda I = L L^T,
//   alpha = L^{-T} L^{-1} Y,  pred = K_test alpha.
//
// Blocked right-looking Cholesky in panels of 64 columns, two launches each:
// the panel (its diagonal block and the rows below it) and the trailing
// update on the float64 matrix cores.  Right-hand sides ride along in the
// same launches (forward substitution); the backward one is a launch per panel.
#include "mfma64.h"

namespace nk {

constexpr int CH_NB = 64;

__global__ __launch_bounds__(256) void krr_diag_mean_kernel(const float* __restrict__ K, int64_t n, int64_t ld,
                                                            double* __restrict__ out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)K[i * ld + i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0] / (double)n;
}

// A = K + (ridge_rel * mean) I   (lower triangle and diagonal are what matter)
__global__ __launch_bounds__(256) void krr_build_kernel(const float* __restrict__ K, int64_t n, const double* mean,
                                                        double ridge_rel, double lam_abs, double* __restrict__ A,
                                                        int* __restrict__ info) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e == 0) info[0] = 0;
  if (e >= n * n) return;
  const int64_t i = e / n, j = e - i * n;
  double v = (double)K[e];
  if (i == j) v = chol_diagonal(v + (ridge_rel >= 0.0 ? ridge_rel * mean[0] : lam_abs));
  A[e] = v;
}

// The factored 64 x 64 diagonal block of a panel in the matrix: L in its
// lower triangle, and in the strict upper triangle of each 16 x 16 block on
// its diagonal the strictly lower part of that block's inverse, transposed.
// With the inverses a triangular solve is a chain of 16 x 16 products for the
// matrix cores.  Blocks of 16 add no error that shows beside the substitution's
// own: on factors of 256 points in groups of 16 that coincide to 1e-3, 1e-4 and
// 1e-6 (condition 1e8 to 1e13) the solutions are as far from an extended
// precision one as LAPACK's (1.0e-9, 3.8e-7 and 9.3e-5 of the largest, LAPACK
// 1.8e-9, 6.9e-7 and 1.7e-4), the residuals too.  In LDS: L in T, the whole
// inverses in V.
constexpr int CH_LD = CH_NB + 1, CH_LV = 17;

struct CholLds {
  double T[CH_NB * CH_LD];
  double V[4 * 16 * CH_LV];
};

// X_b of one 16-column strip for the four 16-row blocks of a panel: X = L^{-1} Y
// (BACK: L^{-T} Y), y[b] in the matrix cores' result layout, in place.
template <bool BACK>
__device__ __forceinline__ void chol_chain(const CholLds& m, d4 (&y)[4]) {
  const int i = threadIdx.x & 15, g = (threadIdx.x >> 4) & 3;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int b = BACK ? 3 - s : s;
    d4 v = y[b];
#pragma unroll
    for (int u = 0; u < s; ++u) {
      const int a = BACK ? 3 - u : u;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = 4 * t + g;
        v = mfma64(BACK ? -m.T[(16 * a + k) * CH_LD + 16 * b + i] : -m.T[(16 * b + i) * CH_LD + 16 * a + k], y[a][t],
                   v);
      }
    }
    d4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = 4 * t + g;
      x = mfma64(m.V[16 * b * CH_LV + (BACK ? k * CH_LV + i : i * CH_LV + k)], v[t], x);
    }
    y[b] = x;
  }
}

// A panel's strip of right-hand sides: rows k + 16 b + 4 t + g, column col.
// (Here as in the other kernels of the factorisation loads are clamped into
// the matrix and what lies past its end is replaced afterwards: loads under a
// condition went out one after another, 12000 of a panel's 52000 cycles.)
__device__ __forceinline__ void chol_load_strip(const double* Z, int64_t n, int64_t k, int64_t c, int64_t col, int g,
                                                d4 (&y)[4]) {
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t r = k + 16 * b + 4 * t + g;
      y[b][t] = Z[(r < n ? r : n - 1) * c + col];
    }
  if (k + CH_NB <= n) return;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (k + 16 * b + 4 * t + g >= n) y[b][t] = 0.0;
}
__device__ __forceinline__ void chol_store_strip(double* Z, int64_t n, int64_t k, int64_t c, int64_t col, int g,
                                                 const d4 (&y)[4]) {
  if (col >= c) return;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t r = k + 16 * b + 4 * t + g;
      if (r < n) Z[r * c + col] = y[b][t];
    }
}

// 1 / d: the hardware's estimate (relative error about 2^-23) and a cubic step.
__device__ __forceinline__ double chol_rcp(double d) {
  const double r = __builtin_amdgcn_rcp(d), e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Panel [k, k + nb): every workgroup factors the diagonal block for itself
// (a launch of its own for it would add to the chain that bounds the solve:
// n columns, one after the other).  The first nrow workgroups solve 64 of the
// rows below each, 16 per wave: A[i, panel] <- A[i, panel] L^{-T}; the others
// 64 right-hand sides each: Z[panel] <- L^{-1} Z[panel].  Workgroup 0 stores
// the factor: into place if it is the only one, else beside it, at columns
// k + 64 .. k + 127 of the unused upper triangle, since the others may still
// be reading the block (chol_update_kernel moves it).
// The columns are factored 16 at a time by one wave, a lane per row of the
// block, pivots and multipliers by lane reads: no barrier inside.  With a
// barrier per column (block in LDS, one workgroup, its own launch) and a
// thread per row below: 82 + 43 us a panel at n = 2500; 23 us for
// both with a square root between pivots and each broadcast read where it is
// used (400 cycles a column) and loads under conditions; 17 us so, of which 2.7
// load, 8.5 factor and update the block, 2.7 invert its last part and solve.
__global__ __launch_bounds__(256) void chol_panel_kernel(double* __restrict__ A, int64_t n, int64_t k, int nb,
                                                         int* __restrict__ info, unsigned nrow,
                                                         double* __restrict__ Z, int64_t c) {
  __shared__ CholLds m;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int64_t rest = n - k - nb;
  const bool rhs = blockIdx.x >= nrow;
  // this wave's 16 rows below or right-hand sides, and the diagonal block
  // (all requested before the first is used)
  const int64_t row = k + nb + (int64_t)blockIdx.x * CH_NB + 16 * w + i;
  const int64_t col = (int64_t)(blockIdx.x - nrow) * 64 + 16 * w + i;
  double* prow = A + (row < n ? row : n - 1) * n + k;
  double dv[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + w;
    dv[q] = A[(k + (r < nb ? r : nb - 1)) * n + k + (lane < nb ? lane : nb - 1)];
  }
  d4 y[4];
  if (rhs) {
    chol_load_strip(Z, n, k, c, col < c ? col : c - 1, g, y);
  } else if (rest > 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) y[b][t] = prow[16 * b + 4 * t + g];
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + w;
    m.T[r * CH_LD + lane] = (r < nb && lane <= r) ? dv[q] : (r == lane ? 1.0 : 0.0);
  }
  __syncthreads();
  // inverse of a diagonal block: lane i forms its column i (wave 3, while wave
  // 0 factors the next block)
  auto inverse = [&](int b) {
    if (g != 0) return;
    const double* L = m.T + 16 * b * CH_LD + 16 * b;
    const double ri = 1.0 / L[i * CH_LD + i];
    double x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = r == i ? 1.0 : 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      x[r] *= lane_value(ri, r);
#pragma unroll
      for (int e = r + 1; e < 16; ++e) x[e] = fma(-L[e * CH_LD + r], x[r], x[e]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) m.V[(16 * b + r) * CH_LV + i] = x[r];  // (0 above the diagonal)
  };
#pragma unroll 1
  for (int jb = 0; jb < 4; ++jb) {
    if (w == 3 && jb > 0) inverse(jb - 1);
    if (w == 0) {
      // (rotated, so that the block's own rows are lanes 0 .. 15)
      const int row = (lane + 16 * jb) & 63;
      double a[16], b[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) a[j] = m.T[row * CH_LD + 16 * jb + j];
      // Column j of the unscaled factor: a[e] -= (a[j] / d) a_e[j], d the
      // pivot.  Between one pivot and the next stand 1 / d (a cubic step on the
      // hardware's estimate), two products and a broadcast; the other columns'
      // updates and the next column's broadcasts (b) pass under them, each
      // kind in one go, since a broadcast read just before its use costs the
      // wave its latency (schedule fixed by the barriers).  The square roots
      // are taken for the 16 columns at once, when all pivots are known.
      double r = chol_rcp(lane_value(a[0], 0));
#pragma unroll
      for (int e = 1; e < 16; ++e) b[e] = lane_value(a[0], e);
#pragma unroll
      for (int j = 0; j < 15; ++j) {
        const double u = -a[j] * r;
        a[j + 1] = fma(u, b[j + 1], a[j + 1]);
        const double d = lane_value(a[j + 1], j + 1);
        const double r0 = __builtin_amdgcn_rcp(d);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = j + 2; e < 16; ++e) a[e] = fma(u, b[e], a[e]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = j + 2; e < 16; ++e) b[e] = lane_value(a[j + 1], e);
        const double e1 = fma(-d, r0, 1.0);
        r = fma(r0, fma(e1, e1, e1), r0);
        __builtin_amdgcn_sched_barrier(0);
      }
      double d = 1.0;  // lane j < 16: pivot j
#pragma unroll
      for (int j = 0; j < 16; ++j) d = lane == j ? a[j] : d;
      // (a pivot that is not positive spoils the columns after it; the caller
      // reports the flag instead of a result)
      if (!(d > 0.0)) info[0] = 1;
      // 1 / sqrt(d) by two Newton steps, sqrt(d) with its residual
      double rs = __builtin_amdgcn_rsq(d);
      rs = fma(0.5 * rs, fma(-d * rs, rs, 1.0), rs);
      rs = fma(0.5 * rs, fma(-d * rs, rs, 1.0), rs);
      double sq = d * rs;
      sq = fma(fma(-sq, sq, d), 0.5 * rs, sq);
#pragma unroll
      for (int j = 0; j < 16; ++j) m.T[row * CH_LD + 16 * jb + j] = lane == j ? sq : a[j] * lane_value(rs, j);
    }
    __syncthreads();
    // the blocks right of it: T[rb][cb] -= L[rb][jb] L[cb][jb]^T, jb < cb <= rb
    int tile = 0;
    for (int rb = jb + 1; rb < 4; ++rb)
      for (int cb = jb + 1; cb <= rb; ++cb, ++tile) {
        if ((tile & 3) != w) continue;
        d4 acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = m.T[(16 * rb + 4 * v + g) * CH_LD + 16 * cb + i];
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc = mfma64(-m.T[(16 * rb + i) * CH_LD + 16 * jb + 4 * t + g],
                       m.T[(16 * cb + i) * CH_LD + 16 * jb + 4 * t + g], acc);
#pragma unroll
        for (int v = 0; v < 4; ++v) m.T[(16 * rb + 4 * v + g) * CH_LD + 16 * cb + i] = acc[v];
      }
    __syncthreads();
  }
  if (w == 3) inverse(3);
  __syncthreads();
  if (blockIdx.x == 0) {
    const int64_t off = rest > CH_NB ? CH_NB : 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int r = 4 * q + w;
      const bool inv = lane > r && (lane >> 4) == (r >> 4);
      const double v = inv ? m.V[lane * CH_LV + (r & 15)] : m.T[r * CH_LD + lane];
      if (r < nb && lane < nb) A[(k + r) * n + k + off + lane] = v;
    }
  }
  if (rhs || rest > 0) {
    chol_chain<false>(m, y);
    if (rhs) {
      chol_store_strip(Z, n, k, c, col, g, y);
    } else if (row < n) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) prow[16 * b + 4 * t + g] = y[b][t];
    }
  }
}

// Trailing update for the 64-column panel at k (base = k + 64): of the matrix,
// A[i][j] -= sum_t A[i][k + t] A[j][k + t], base <= j <= i < n, one 64 x 64 tile
// of the lower triangle per workgroup and a 32 x 32 quadrant per wave
// (blocks [0, ntiles)); of the right-hand sides, Z[i] -= sum_t A[i][k + t]
// Z[k + t], 64 rows of one strip per workgroup (the last nrhs blocks); and one
// block moves the panel's factor into place (move).  All operands of a tile
// are requested at once, straight from the caches: at the sizes solved here a
// launch is a few tiles per CU, bound by one round of latency (45 -> 12 us
// a panel at n = 2500 against dot products on the vector unit from LDS), and by
// HBM traffic of the tile itself beyond.
__global__ __launch_bounds__(256) void chol_update_kernel(double* __restrict__ A, int64_t n, int64_t k,
                                                          unsigned ntiles, int move, double* __restrict__ Z,
                                                          int64_t c, unsigned nbk) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int64_t base = k + CH_NB;
  if (blockIdx.x >= ntiles) {
    if (move && blockIdx.x == ntiles) {
      double v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = A[(k + 4 * q + w) * n + base + lane];
#pragma unroll
      for (int q = 0; q < 16; ++q) A[(k + 4 * q + w) * n + k + lane] = v[q];
      return;
    }
    const unsigned e = blockIdx.x - ntiles - move;
    const int64_t j0 = (int64_t)(e / nbk) * 16, r0 = base + (int64_t)(e % nbk) * 64 + 16 * w;
    const int64_t col = j0 + i < c ? j0 + i : c - 1;
    const double* pa = A + (r0 + i < n ? r0 + i : n - 1) * n + k + 4 * g;
    double a[4][4], b[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      load4(pa + 16 * q, a[q]);
#pragma unroll
      for (int t = 0; t < 4; ++t) b[q][t] = Z[(k + 16 * q + 4 * g + t) * c + col];
    }
    d4 acc;
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = Z[(r0 + 4 * v + g < n ? r0 + 4 * v + g : n - 1) * c + col];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc = mfma64(-a[q][t], b[q][t], acc);
    if (j0 + i < c) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (r0 + 4 * v + g < n) Z[(r0 + 4 * v + g) * c + col] = acc[v];
    }
    return;
  }
  int64_t bi = (int64_t)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
  while (bi * (bi + 1) / 2 > (int64_t)blockIdx.x) --bi;
  while ((bi + 1) * (bi + 2) / 2 <= (int64_t)blockIdx.x) ++bi;
  const int64_t bj = (int64_t)blockIdx.x - bi * (bi + 1) / 2;
  const int64_t r0 = base + 64 * bi + 32 * (w >> 1), c0 = base + 64 * bj + 32 * (w & 1);
  if (c0 > r0 || r0 >= n) return;  // the quadrant above the diagonal, or past the end
  double av[2][4][4], bv[2][4][4];
  d4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int64_t ra = r0 + 16 * x + i, rb = c0 + 16 * x + i;
    const double* pa = A + (ra < n ? ra : n - 1) * n + k + 4 * g;
    const double* pb = A + (rb < n ? rb : n - 1) * n + k + 4 * g;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      load4(pa + 16 * q, av[x][q]);
      load4(pb + 16 * q, bv[x][q]);
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int64_t cc = c0 + 16 * y + i;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + 16 * x + 4 * v + g;
        acc[x][y][v] = A[(r < n ? r : n - 1) * n + (cc < n ? cc : n - 1)];
      }
    }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = mfma64(-av[x][q][t], bv[y][q][t], acc[x][y]);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int64_t cc = c0 + 16 * y + i;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + 16 * x + 4 * v + g;
        if (r < n && cc <= r) A[r * n + cc] = acc[x][y][v];
      }
    }
}

// One panel of a substitution with the factor in A: X[panel] = L_pp^{-1}
// Z[panel] (BACK: L_pp^{-T}) and the products with it taken off the rows not
// yet solved, 64 of them (tile) for one strip of 16 columns per workgroup;
// every wave solves the panel's strip for itself (a chain of 40 products,
// about a microsecond) so that a panel is one launch.  X is another array
// than Z when there are tiles: the others may still be reading Z's panel.
template <bool BACK>
__global__ __launch_bounds__(256) void chol_solve_kernel(const double* __restrict__ A, int64_t n, int64_t k,
                                                         double* Z, int64_t c, double* X, unsigned ntiles) {
  __shared__ CholLds m;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const unsigned per = ntiles > 0 ? ntiles : 1, strip = blockIdx.x / per, tile = blockIdx.x - strip * per;
  const int64_t j0 = (int64_t)strip * 16, col = j0 + i < c ? j0 + i : c - 1;
  const int64_t r0 = (BACK ? 0 : k + CH_NB) + (int64_t)tile * 64 + 16 * w;
  double f[16], a[4][4];
  d4 y[4], acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + w;
    f[q] = A[(k + r < n ? k + r : n - 1) * n + (k + lane < n ? k + lane : n - 1)];
  }
  chol_load_strip(Z, n, k, c, col, g, y);
  if (ntiles > 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t kk = k + 16 * b + 4 * t + g, r = r0 + i;
        // (backward: rows of the panel, past the end in the last one; forward: rows below)
        if (BACK)
          a[b][t] = A[(kk < n ? kk : n - 1) * n + r];
        else
          a[b][t] = A[(r < n ? r : n - 1) * n + kk];
      }
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = Z[(r0 + 4 * v + g < n ? r0 + 4 * v + g : n - 1) * c + col];
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = 4 * q + w, rb = r & 15, lb = lane & 15;
    if (k + r >= n || k + lane >= n) f[q] = r == lane ? 1.0 : 0.0;
    m.T[r * CH_LD + lane] = f[q];
    if ((lane >> 4) == (r >> 4)) {
      // upper triangle: the inverse, transposed; it is 0 above its diagonal
      if (lane >= r) m.V[lane * CH_LV + rb] = lane == r ? 1.0 / f[q] : f[q];
      if (lane > r) m.V[r * CH_LV + lb] = 0.0;
    }
  }
  __syncthreads();
  chol_chain<BACK>(m, y);
  if (tile == 0 && w == 0) chol_store_strip(X, n, k, c, j0 + i, g, y);
  if (ntiles > 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc = mfma64(-a[b][t], y[b][t], acc);
    if (j0 + i < c) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (r0 + 4 * v + g < n) Z[(r0 + 4 * v + g) * c + col] = acc[v];
    }
  }
}

// resid = G - Y_t with G = K_ts alpha (m x c) on entry; G = 2 resid / (m c); sq = resid^2
__global__ __launch_bounds__(256) void krr_resid_kernel(int64_t mc, const float* __restrict__ Yt,
                                                        double* __restrict__ G, double* __restrict__ sq) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= mc) return;
  const double r = G[e] - (double)Yt[e];
  G[e] = 2.0 * r / (double)mc;
  sq[e] = r * r;
}

// loss = sum(sq) / count, fixed-order reduction in one workgroup
__global__ __launch_bounds__(256) void krr_loss_kernel(const double* __restrict__ sq, int64_t cnt,
                                                       double* __restrict__ loss) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t e = threadIdx.x; e < cnt; e += 256) s += sq[e];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = red[0] / (double)cnt;
}

// out (rows x cols, float) = scale * U V^T with U (rows x c), V (cols x c) double
__global__ __launch_bounds__(256) void krr_outer_kernel(const double* __restrict__ U, int64_t rows,
                                                        const double* __restrict__ V, int64_t cols, int64_t c,
                                                        double scale, float* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= rows * cols) return;
  const int64_t i = e / cols, t = e - i * cols;
  double s = 0.0;
  for (int64_t k = 0; k < c; ++k) s += U[i * c + k] * V[t * c + k];
  out[e] = (float)(scale * s);
}

int launch_krr_mse_bwd(const float* Kts, int64_t m, int64_t n, const double* alpha, int64_t c, const float* Yt,
                       double* G, double* sq, double* loss, double* B, hipStream_t s) {
  if (dn_gemm_fd(Kts, n, false, alpha, c, G, c, m, c, n, 1.0, 0.0, false, s)) return -3;
  hipLaunchKernelGGL(krr_resid_kernel, dim3((unsigned)((m * c + 255) / 256)), dim3(256), 0, s, m * c, Yt, G, sq);
  hipLaunchKernelGGL(krr_loss_kernel, dim3(1), dim3(256), 0, s, sq, m * c, loss);
  return dn_gemm_fd(Kts, n, true, G, c, B, c, n, c, m, 1.0, 0.0, false, s);
}

int launch_krr_outer(const double* U, int64_t rows, const double* V, int64_t cols, int64_t c, double scale,
                     float* out, hipStream_t s) {
  hipLaunchKernelGGL(krr_outer_kernel, dim3((unsigned)((rows * cols + 255) / 256)), dim3(256), 0, s, U, rows, V, cols,
                     c, scale, out);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template <bool BACK>
static void chol_solve_launch(const double* A, int64_t n, int64_t k, double* Z, int64_t c, double* X, int64_t ntiles,
                              hipStream_t s) {
  const int64_t strips = (c + 15) / 16;
  hipLaunchKernelGGL(chol_solve_kernel<BACK>, dim3((unsigned)(strips * (ntiles > 0 ? ntiles : 1))), dim3(256), 0, s, A,
                     n, k, Z, c, X, (unsigned)ntiles);
}

int launch_cholesky(double* A, int64_t n, int* info, double* Z, int64_t c, hipStream_t s) {
  if (!Z) c = 0;
  for (int64_t k = 0; k < n; k += CH_NB) {
    const int nb = (int)((n - k) < CH_NB ? (n - k) : CH_NB);
    const int64_t rest = n - k - nb, nbk = (rest + CH_NB - 1) / CH_NB;
    // (with at most one workgroup of rows the factor goes straight into place,
    // and the right-hand sides follow in a launch of their own)
    const bool ride = c > 0 && rest > CH_NB;
    const unsigned nrow = (unsigned)(nbk > 0 ? nbk : 1);
    hipLaunchKernelGGL(chol_panel_kernel, dim3(nrow + (ride ? (unsigned)((c + 63) / 64) : 0)), dim3(256), 0, s, A, n, k,
                       nb, info, nrow, Z, c);
    if (c > 0 && !ride) chol_solve_launch<false>(A, n, k, Z, c, Z, 0, s);
    if (rest > 0) {
      const int64_t ntiles = nbk * (nbk + 1) / 2;
      const int move = rest > CH_NB ? 1 : 0;
      hipLaunchKernelGGL(chol_update_kernel, dim3((unsigned)(ntiles + move + (c + 15) / 16 * nbk)), dim3(256), 0, s, A,
                         n, k, (unsigned)ntiles, move, Z, c, (unsigned)nbk);
    }
  }
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_chol_forward(const double* A, int64_t n, double* Z, int64_t c, double* X, hipStream_t s) {
  if (n <= 0 || c <= 0) return 0;
  for (int64_t k = 0; k < n; k += CH_NB)
    chol_solve_launch<false>(A, n, k, Z, c, X, n - k > CH_NB ? (n - k - 1) / CH_NB : 0, s);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_chol_backward(const double* A, int64_t n, double* Z, int64_t c, double* X, hipStream_t s) {
  if (n <= 0 || c <= 0) return 0;
  for (int64_t k = (n - 1) / CH_NB * CH_NB; k >= 0; k -= CH_NB) chol_solve_launch<true>(A, n, k, Z, c, X, k / CH_NB, s);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_krr_build(const float* K, int64_t n, double ridge_rel, double lam_abs, double* mean, double* A,
                     int* info, hipStream_t s) {
  if (ridge_rel >= 0.0) hipLaunchKernelGGL(krr_diag_mean_kernel, dim3(1), dim3(256), 0, s, K, n, n, mean);
  hipLaunchKernelGGL(krr_build_kernel, dim3((unsigned)((n * n + 255) / 256)), dim3(256), 0, s, K, n, mean,
                     ridge_rel, lam_abs, A, info);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace nk
