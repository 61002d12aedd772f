// Kernel regression by preconditioned conjugate gradients in float64
// (Sec. 2, "Iterative solvers": CG with the partial pivoted Cholesky
// preconditioner; Sec. 1, related work: the preconditioner's origin and the
// need for high precision on neural kernels).
//
// System (K + lam I) X = Y, K the float32 Gram matrix the kernel entry points
// write (n x n, leading dim ldk, row-major, symmetric), Y and X float64
// (n x c).  Every product and sum runs in float64 on the float32 values of
// K, so the system solved is exactly double(K) + lam I.
//
// Pieces:
//   * pchol_*: greedy partial pivoted Cholesky K ~ L L^T (L n x r, column
//     major), one kernel per pivot: every workgroup reduces the previous
//     step's per-workgroup maxima of the residual diagonal d (largest value,
//     lowest index on ties), then forms its rows of the new column and
//     updates d.  Picked indices hold d = -inf.
//   * The preconditioner Ph = L L^T + lam I is applied with the Woodbury
//     identity Ph^{-1} v = (v - L M^{-1} L^T v) / lam, M = lam I + L^T L.
//     With M = R R^T (Cholesky) and U = L R^{-T}, formed once in place of L
//     by a forward substitution (a row-major copy is what the products read), this is (v - U (U^T v)) / lam: two
//     skinny products per application and an operator that stays symmetric
//     in floating point (an explicitly inverted M does not, and CG then
//     stalls above small tolerances).
//   * kmv_*: Q = (K + lam I) P, the product that dominates each iteration:
//     K is streamed once from HBM as float4 rows.  Because K is symmetric,
//     Q[i] = sum_j K[j][i] P[j]: a workgroup owns 256 columns, lane l of each
//     of its four waves columns 4l..4l+3, and the waves walk every fourth
//     group of four rows j of the row split; P[j][:] is the same for the whole
//     wave, so it arrives through scalar loads and feeds the FMAs as a scalar
//     operand.  The waves meet in LDS; row splits write partial sums, reduced
//     in a fixed order by the next kernel (which also adds lam P and the
//     per-workgroup partials of p.q).
//   * CG vector steps, 64 rows of all columns per workgroup, one thread per
//     element; every dot product is reduced in a fixed order (per-workgroup
//     partials, summed again by each workgroup that needs the total), so
//     results are reproducible.  Per-column state (gamma, active flag,
//     iteration count, relative residual) lives in device memory, gamma and
//     the flags in two copies (an iteration reads one and writes the other, so
//     that no launch is spent on the state alone); a column that meets the
//     tolerance is frozen (alpha = beta = 0 from then on).
//   * The preconditioner's two skinny products run on the float64 matrix cores.
// An iteration of 8192 rows, 10 columns and rank 256 took 173 us in 9 launches
// and a copy (kernel-vector product 58 and its reduction 23, U^T r 22, U w 32)
// and takes about 102 us in 7.
#include <float.h>
#include <limits.h>

#include "mfma64.h"

namespace nk {

constexpr int PC_TPB = 256;
constexpr double kNegInf = -__builtin_huge_val();

__device__ __forceinline__ bool pc_better(double v, int i, double bv, int bi) {
  return v > bv || (v == bv && i < bi);
}

// Deterministic (value, index) maximum over a 256-thread workgroup.
__device__ inline void pc_block_argmax(double& v, int& i) {
  __shared__ double sv[PC_TPB];
  __shared__ int si[PC_TPB];
  const int t = threadIdx.x;
  sv[t] = v;
  si[t] = i;
  __syncthreads();
  for (int w = PC_TPB / 2; w >= 1; w >>= 1) {
    if (t < w && pc_better(sv[t + w], si[t + w], sv[t], si[t])) {
      sv[t] = sv[t + w];
      si[t] = si[t + w];
    }
    __syncthreads();
  }
  v = sv[0];
  i = si[0];
  __syncthreads();
}

// Fixed-order column sums by the PC_TPB threads of a workgroup: out[c] =
// sum_b part[b][c] (b < nb, c < C), through `red` (PC_TPB x C doubles of
// LDS); every thread sees out after the call.
template <int C>
__device__ inline void pc_colsum(const double* __restrict__ part, int nb, double* red, double* out) {
  const int t = threadIdx.x;
  double acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0;
  for (int b = t; b < nb; b += PC_TPB) {
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] += part[(int64_t)b * C + c];
  }
#pragma unroll
  for (int c = 0; c < C; ++c) red[t * C + c] = acc[c];
  __syncthreads();
  for (int w = PC_TPB / 2; w >= 1; w >>= 1) {
    if (t < w) {
#pragma unroll
      for (int c = 0; c < C; ++c) red[t * C + c] += red[(t + w) * C + c];
    }
    __syncthreads();
  }
  if (t < C) out[t] = red[t];
  __syncthreads();
}

// Rows of the n x C vectors per workgroup of the vector steps, PC_ROWS * C
// elements walked by PC_TPB threads in the order they lie in memory.
constexpr int PC_ROWS = 64;

// Fixed-order column sums of a workgroup's PC_ROWS x C products v (LDS, row
// by row), to out[0..C) (global); red: 16 x C doubles of LDS.
template <int C>
__device__ inline void pc_block_sums(const double* v, double* red, double* __restrict__ out) {
  const int t = threadIdx.x;
  __syncthreads();
  if (t < 16 * C) {
    const int q = t / C, c = t - q * C;
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < PC_ROWS / 16; ++r) s += v[(q * (PC_ROWS / 16) + r) * C + c];
    red[t] = s;
  }
  __syncthreads();
  if (t < C) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) s += red[q * C + t];
    out[t] = s;
  }
}

// Fixed-order block sum of one value per thread, written to out (thread 0).
__device__ inline void pc_block_sum_store(double v, double* out) {
  __shared__ double red[PC_TPB];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = PC_TPB / 2; w >= 1; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
  __syncthreads();
}

// d = diag(K); per-workgroup maximum of d.
__global__ __launch_bounds__(PC_TPB) void pchol_init_kernel(const float* __restrict__ K, int64_t n, int64_t ldk,
                                                            double* __restrict__ d, double* __restrict__ pv,
                                                            int* __restrict__ pi) {
  const int64_t i = (int64_t)blockIdx.x * PC_TPB + threadIdx.x;
  double v = -DBL_MAX;
  int idx = INT_MAX;
  if (i < n) {
    v = (double)K[i * ldk + i];
    d[i] = v;
    idx = (int)i;
  }
  pc_block_argmax(v, idx);
  if (threadIdx.x == 0) {
    pv[blockIdx.x] = v;
    pi[blockIdx.x] = idx;
  }
}

// Pivot step m: column m of L (column major, leading dim n) and the update of
// d.  A step is a chain of a reduction, a gather and a sum over the earlier
// columns, and n / ROWS workgroups wide.  ROWS = 64: the four waves sum a
// quarter of the columns each (9.0 us a step at n = 8192 and up to 256 columns
// with 256 rows and one thread walking all of them, 6.4 us now); ROWS = 256
// for a workspace that holds maxima for that many workgroups only.
constexpr int PV_TPB = PC_TPB;

// Maximum (value, lowest index) over the workgroup, in every thread.
__device__ inline void pv_argmax(double& v, int& i) {
  __shared__ double sv[PV_TPB / 64];
  __shared__ int si[PV_TPB / 64];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double ov = __shfl_xor(v, off);
    const int oi = __shfl_xor(i, off);
    if (pc_better(ov, oi, v, i)) {
      v = ov;
      i = oi;
    }
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = v;
    si[threadIdx.x >> 6] = i;
  }
  __syncthreads();
  v = sv[0];
  i = si[0];
#pragma unroll
  for (int w = 1; w < PV_TPB / 64; ++w)
    if (pc_better(sv[w], si[w], v, i)) {
      v = sv[w];
      i = si[w];
    }
}

template <int ROWS>
__global__ __launch_bounds__(PV_TPB) void pchol_step_kernel(const float* __restrict__ K, int64_t n, int64_t ldk,
                                                            double* __restrict__ L, int m, double* __restrict__ d,
                                                            const double* __restrict__ pv_in,
                                                            const int* __restrict__ pi_in, int nb,
                                                            double* __restrict__ pv_out, int* __restrict__ pi_out,
                                                            int* __restrict__ piv, double* __restrict__ dpiv,
                                                            double pivot_tol) {
  extern __shared__ double lp[];  // L[p][0..m), then the quarters' sums
  double* quarter = lp + m;
  constexpr int PARTS = PV_TPB / ROWS;
  const int t = threadIdx.x, row = t & (ROWS - 1), part = t / ROWS;
  double v = -DBL_MAX;
  int idx = INT_MAX;
  for (int b = t; b < nb; b += PV_TPB) {
    if (pc_better(pv_in[b], pi_in[b], v, idx)) {
      v = pv_in[b];
      idx = pi_in[b];
    }
  }
  pv_argmax(v, idx);
  const double dmax = v;
  const int p = idx;
  const double dmax0 = m == 0 ? dmax : dpiv[0];
  const int64_t i = (int64_t)blockIdx.x * ROWS + row;
  if (!(dmax > 0.0) || dmax <= pivot_tol * dmax0 || p >= n) {
    // rank reached: zero column, and pass the same maximum on so that every
    // later step stops too
    if (i < n && part == 0) L[(int64_t)m * n + i] = 0.0;
    if (t == 0) {
      pv_out[blockIdx.x] = dmax;
      pi_out[blockIdx.x] = p;
      if (blockIdx.x == 0) {
        piv[m] = -1;
        dpiv[m] = 0.0;
      }
    }
    return;
  }
  for (int k = t; k < m; k += PV_TPB) lp[k] = L[(int64_t)k * n + p];
  double kp = 0.0, di = 0.0;
  if (i < n && part == 0) {
    kp = (double)K[(int64_t)p * ldk + i];
    di = d[i];
  }
  __syncthreads();
  const int k0 = (int)((int64_t)m * part / PARTS), k1 = (int)((int64_t)m * (part + 1) / PARTS);
  double acc = 0.0;
  if (i < n) {
#pragma unroll 8
    for (int k = k0; k < k1; ++k) acc = fma(L[(int64_t)k * n + i], lp[k], acc);
  }
  if (part > 0) quarter[(part - 1) * ROWS + row] = acc;
  __syncthreads();
  double nv = -DBL_MAX;
  int nidx = INT_MAX;
  if (i < n && part == 0) {
    const double sp = sqrt(dmax);
    double l;
    if (i == p) {
      l = sp;
      di = kNegInf;
    } else if (di == kNegInf) {
      l = 0.0;
    } else {
#pragma unroll
      for (int q = 1; q < PARTS; ++q) acc += quarter[(q - 1) * ROWS + row];
      l = (kp - acc) / sp;
      di -= l * l;
    }
    L[(int64_t)m * n + i] = l;
    d[i] = di;
    nv = di;
    nidx = (int)i;
  }
  pv_argmax(nv, nidx);
  if (t == 0) {
    pv_out[blockIdx.x] = nv;
    pi_out[blockIdx.x] = nidx;
    if (blockIdx.x == 0) {
      piv[m] = p;
      dpiv[m] = dmax;
    }
  }
}

template <int ROWS>
static int pchol_steps(const float* K, int64_t n, int64_t ldk, int rank, double pivot_tol, double* L, int* piv,
                       double* d, double* pv, int* pi, double* dpiv, hipStream_t s) {
  static std::atomic<size_t> seen[kMaxDevices];
  const int nb0 = (int)((n + PC_TPB - 1) / PC_TPB), nb = (int)((n + ROWS - 1) / ROWS);
  hipLaunchKernelGGL(pchol_init_kernel, dim3(nb0), dim3(PC_TPB), 0, s, K, n, ldk, d, pv, pi);
  for (int m = 0; m < rank; ++m) {
    const int a = m & 1, b = a ^ 1;
    const size_t lds = (size_t)(m + PC_TPB) * sizeof(double);
    if (allow_dyn_lds((const void*)pchol_step_kernel<ROWS>, lds, seen)) return -3;
    hipLaunchKernelGGL(pchol_step_kernel<ROWS>, dim3(nb), dim3(PV_TPB), lds, s, K, n, ldk, L, m, d,
                       pv + (size_t)a * nb, pi + (size_t)a * nb, m == 0 ? nb0 : nb, pv + (size_t)b * nb,
                       pi + (size_t)b * nb, piv, dpiv, pivot_tol);
  }
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_pchol(const float* K, int64_t n, int64_t ldk, int rank, double pivot_tol, double* L, int* piv,
                 double* d, double* pv, int* pi, int64_t maxima, double* dpiv, hipStream_t s) {
  return maxima >= (n + 63) / 64 ? pchol_steps<64>(K, n, ldk, rank, pivot_tol, L, piv, d, pv, pi, dpiv, s)
                                 : pchol_steps<256>(K, n, ldk, rank, pivot_tol, L, piv, d, pv, pi, dpiv, s);
}

// ---- preconditioner set-up ----------------------------------------------

// Lr (n x r, row major) <- L (n x r, column major)
__global__ __launch_bounds__(PC_TPB) void pc_transpose_kernel(const double* __restrict__ L, int64_t n, int r,
                                                              double* __restrict__ Lr) {
  __shared__ double tile[32][33];
  const int64_t i0 = (int64_t)blockIdx.x * 32;
  const int a0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int y = ty; y < 32; y += 8) {
    const int a = a0 + y;
    const int64_t i = i0 + tx;
    tile[y][tx] = (a < r && i < n) ? L[(int64_t)a * n + i] : 0.0;
  }
  __syncthreads();
  for (int y = ty; y < 32; y += 8) {
    const int64_t i = i0 + y;
    const int a = a0 + tx;
    if (a < r && i < n) Lr[i * r + a] = tile[tx][y];
  }
}

int launch_pc_setup(double* LU, int64_t n, int r, double lam, double* Ur, double* M, int* info, hipStream_t s) {
  if (r == 0) return 0;
  // M = lam I + L^T L.  The Woodbury form subtracts L M^{-1} L^T from the
  // identity, which along the leading directions of K leaves only about
  // lam / sigma^2 (sigma^2 up to the largest eigenvalue of K): so M has to
  // match L^T L to about one rounding of its entries, or the preconditioner
  // loses definiteness there and CG stalls.  A plain running sum over n rows
  // is off by up to n roundings; the product is compensated.
  if (dn_ltl(LU, n, r, lam, M, info, s)) return -3;
  // U = L R^{-T} in place: with L stored column major (an r x n row-major
  // array), U^T = R^{-1} L^T is a forward substitution with n right-hand
  // sides, which ride along in the factorisation of M
  if (launch_cholesky(M, r, info, LU, n, s)) return -3;
  hipLaunchKernelGGL(pc_transpose_kernel, dim3((unsigned)((n + 31) / 32), (unsigned)((r + 31) / 32)), dim3(PC_TPB),
                     0, s, LU, n, r, Ur);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// ---- Q = (K + lam I) P ----------------------------------------------------

constexpr int KMV_COLS = 256;  // columns of K per workgroup (64 lanes x 4)
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A kernel of a conjugate-gradient iteration returns at once when its gate
// (the solver's "some column still iterates" flag) reads 0.
#define NK_PCG_GATE(g) \
  if ((g) != nullptr && *(g) == 0) return;

// Partial sums over rows [j0, j1) of K for the 256 columns of this block:
// part[s][i][c] = sum_j K[j][i] P[j][c].
template <int C, bool VEC>
__global__ __launch_bounds__(PC_TPB) void kmv_partial_kernel(const float* __restrict__ K, int64_t n, int64_t ldk,
                                                             const double* __restrict__ P, int64_t rows_per_split,
                                                             double* __restrict__ part, const int* __restrict__ gate) {
  NK_PCG_GATE(gate)
  __shared__ double red[2][4 * C][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (int64_t)blockIdx.x * KMV_COLS + 4 * lane;
  const int64_t j0 = (int64_t)blockIdx.y * rows_per_split;
  const int64_t j1 = j0 + rows_per_split < n ? j0 + rows_per_split : n;
  double acc[4][C];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[e][c] = 0.0;
  auto add_row = [&](const float (&kv)[4], int64_t j) {
    const double* pr = P + j * C;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double kd = (double)kv[e];
#pragma unroll
      for (int c = 0; c < C; ++c) acc[e][c] = fma(kd, pr[c], acc[e][c]);
    }
  };
  if (i0 < n) {
    // four rows per step, the next step's loads issued before this one's
    // FMAs; K is read once per product, so its loads are non-temporal (they
    // do not evict P from the caches)
    const float* kb = K + i0;
    int64_t j = j0 + 4 * w;
    auto fetch = [&](float (&kv)[4][4], int64_t row) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (VEC) {
          const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(kb + (row + u) * ldk));
          kv[u][0] = t.x;
          kv[u][1] = t.y;
          kv[u][2] = t.z;
          kv[u][3] = t.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) kv[u][e] = i0 + e < n ? kb[(row + u) * ldk + e] : 0.f;
        }
      }
    };
    float even[4][4], odd[4][4];
    // (past the last step: its own rows again, in bounds and not used)
    if (j + 4 <= j1) fetch(even, j);
    while (j + 4 <= j1) {
      const bool two = j + 20 <= j1;
      fetch(odd, two ? j + 16 : j);
#pragma unroll
      for (int u = 0; u < 4; ++u) add_row(even[u], j + u);
      j += 16;
      if (!two) break;
      fetch(even, j + 20 <= j1 ? j + 16 : j);
#pragma unroll
      for (int u = 0; u < 4; ++u) add_row(odd[u], j + u);
      j += 16;
    }
    for (; j < j1; ++j) {  // (the wave whose four rows straddle the end)
      float kv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) kv[e] = i0 + e < n ? kb[j * ldk + e] : 0.f;
      add_row(kv, j);
    }
  }
  // waves 2, 3 into 0, 1, then 1 into 0
#pragma unroll
  for (int h = 2; h >= 1; h >>= 1) {
    __syncthreads();
    if (w >= h && w < 2 * h) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < C; ++c) red[w - h][e * C + c][lane] = acc[e][c];
    }
    __syncthreads();
    if (w < h) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < C; ++c) acc[e][c] += red[w][e * C + c][lane];
    }
  }
  if (w != 0) return;
  double* out = part + (int64_t)blockIdx.y * n * C;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (i0 + e < n) {
#pragma unroll
      for (int c = 0; c < C; ++c) out[(i0 + e) * C + c] = acc[e][c];
    }
  }
}

// Q[i] = sum_s part[s][i] + lam P[i]; per-workgroup partials of p.q per column.
template <int C>
__global__ __launch_bounds__(PC_TPB) void kmv_reduce_kernel(const double* __restrict__ part, int S, int64_t n,
                                                            const double* __restrict__ P, double lam,
                                                            double* __restrict__ Q, double* __restrict__ pq_part,
                                                            const int* __restrict__ gate) {
  NK_PCG_GATE(gate)
  __shared__ double prod[PC_ROWS * C], red[16 * C];
  const int64_t e0 = (int64_t)blockIdx.x * PC_ROWS * C, lim = n * C;
#pragma unroll
  for (int x = threadIdx.x; x < PC_ROWS * C; x += PC_TPB) {
    const int64_t e = e0 + x;
    double d = 0.0;
    if (e < lim) {
      double q = 0.0;
#pragma unroll 8
      for (int s = 0; s < S; ++s) q += part[s * lim + e];
      const double p = P[e];
      q = fma(lam, p, q);
      Q[e] = q;
      d = p * q;
    }
    prod[x] = d;
  }
  pc_block_sums<C>(prod, red, pq_part + (int64_t)blockIdx.x * C);
}

// Room for row splits of 16 columns in a workspace (callers keep workspaces, so it
// stays what it has been).
int kmv_splits(int64_t n) {
  const int64_t ncb = (n + KMV_COLS - 1) / KMV_COLS;
  const int64_t most = (n + 63) / 64 < 64 ? (n + 63) / 64 : 64;
  const int64_t S = ((n >= 12288 ? 1024 : 512) + ncb - 1) / ncb;
  return (int)(S > most ? most : S);
}

// Row splits of the product of C columns, at least 64 rows each.  All its
// workgroups take the same time, so what counts is that they fill every CU with
// the same number of them that it holds at once: `per`, and rather one too few
// than one over.  Workgroups per CU and us, 10 columns: n = 12288 1.88 118, 2.06
// 123, 3.0 107, 3.94 115; n = 20000 1.85 299, 2.78 261, 3.7 267, 4.01 326; n = 24576
// 1.88 446, 3.0 376, 3.75 395, 4.12 457; 16 columns (two fit, by registers), n =
// 24576: 1.88 540, 2.25 699, 3.0 591, 3.75 536; one column, n = 20000: 1.85 230, 2.16
// 273, 2.78 234.  Up to 7 columns two are as good as three and write less partial
// sums, and up to 8192 rows for all (n = 5000, 10 columns: 34 and 40; 8192: 58 and
// 60).  Where `per` of them leave more than a tenth empty (n = 36000, 141 column
// blocks: 1.65 of two) a larger number that the columns allow: 16 columns there
// 1257 -> 1125, 4 columns 836 -> 755.
static int kmv_splits(int64_t n, int C) {
  constexpr int64_t cus = 256;
  const int64_t ncb = (n + KMV_COLS - 1) / KMV_COLS, room = (int64_t)kmv_splits(n) * 16 / C;
  // (10 columns are the most of which four fit: where four divide without rest
  // they take 662 us against 683 at n = 32768, 179 against 180 at 16384)
  const bool four = C == 10 && 4 * cus % ncb == 0;
  int per = C >= 8 && C <= 13 && n > 8192 ? (four ? 4 : 3) : 2;
  if (per * cus / ncb > room) per = 2;  // (12 and 13 columns up to 12287 rows)
  const int last = C >= 11 && C <= 13 ? 6 : 4, step = C >= 14 ? 2 : (C >= 11 ? 3 : 1);  // (of 11 to 13 three fit)
  int64_t S = 0, q = 1;  // q workgroups a CU, of which S ncb / (q cus) are there
  for (int p = per; p <= last; p += step) {
    const int64_t s = p * cus / ncb;
    if (S > 0 && s > room) {  // (13 columns, 70000 rows: two splits fill 0.71, 4314 us; the four of the room 3878)
      if (4 * S * ncb < 3 * q * cus) S = room;
      break;
    }
    if (S == 0 || 10 * s * q > 11 * S * p) {
      S = s;
      q = p;
    }
  }
  const int64_t most = (n + 63) / 64 < 64 ? (n + 63) / 64 : 64;
  return (int)(S < 1 ? 1 : (S > most ? most : S));
}

template <int C>
int launch_kmv_c(const float* K, int64_t n, int64_t ldk, const double* P, double lam, double* part, double* Q,
                 double* pq_part, const int* gate, hipStream_t s, ProfHook* hook) {
  const int S = kmv_splits(n, C);
  const int64_t rows = (n + S - 1) / S;
  const bool vec = (ldk % 4 == 0) && ((reinterpret_cast<uintptr_t>(K) & 15) == 0);
  const dim3 grid((unsigned)((n + KMV_COLS - 1) / KMV_COLS), (unsigned)S);
  if (hook) hook->begin(s);
  if (vec)
    hipLaunchKernelGGL((kmv_partial_kernel<C, true>), grid, dim3(PC_TPB), 0, s, K, n, ldk, P, rows, part, gate);
  else
    hipLaunchKernelGGL((kmv_partial_kernel<C, false>), grid, dim3(PC_TPB), 0, s, K, n, ldk, P, rows, part, gate);
  if (hook) hook->end(s);
  hipLaunchKernelGGL((kmv_reduce_kernel<C>), dim3((unsigned)((n + PC_ROWS - 1) / PC_ROWS)), dim3(PC_TPB), 0, s, part,
                     S, n, P, lam, Q, pq_part, gate);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// ---- CG vector steps ------------------------------------------------------

// Per-column state of a CG pass.  Copy k of the doubled entries starts at
// 16 k: an iteration reads copy `it & 1` and its last kernel writes the other.
struct PcgState {
  double* gamma;   // [2][16] r.z of the current residual
  double* ynorm;   // ||y||
  double* relres;  // ||r|| / ||y|| at the column's last update
  int* active;     // [2][16] 1 while the column iterates
  int* iters;      // updates taken
  int* any;        // [2] 1 while some column iterates (the gate of every iteration kernel)
};

// R = Y[:, c0:c0+C], X = 0; partials of ||y||^2.
template <int C>
__global__ __launch_bounds__(PC_TPB) void pcg_init_kernel(const double* __restrict__ Y, int64_t ldy, int64_t c0,
                                                          int64_t n, double* __restrict__ R, double* __restrict__ X,
                                                          double* __restrict__ yy_part) {
  __shared__ double prod[PC_ROWS * C], red[16 * C];
  const int64_t i0 = (int64_t)blockIdx.x * PC_ROWS;
#pragma unroll
  for (int x = threadIdx.x; x < PC_ROWS * C; x += PC_TPB) {
    const int64_t i = i0 + x / C;
    const int c = x % C;
    double y = 0.0;
    if (i < n) {
      y = Y[i * ldy + c0 + c];
      R[i * C + c] = y;
      X[i * C + c] = 0.0;
    }
    prod[x] = y * y;
  }
  pc_block_sums<C>(prod, red, yy_part + (int64_t)blockIdx.x * C);
}

template <int C>
__global__ __launch_bounds__(PC_TPB) void pcg_init_state_kernel(const double* __restrict__ yy_part, int nb,
                                                                PcgState st) {
  __shared__ double red[PC_TPB * C];
  __shared__ double sum[C];
  pc_colsum<C>(yy_part, nb, red, sum);
  const int c = threadIdx.x;
  if (c < C) {
    const double yn = sqrt(sum[c]);
    st.ynorm[c] = yn;
    st.active[c] = yn > 0.0 ? 1 : 0;
    st.iters[c] = 0;
    st.relres[c] = yn > 0.0 ? 1.0 : 0.0;
    sum[c] = yn;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int a = 0;
    for (int k = 0; k < C; ++k) a |= sum[k] > 0.0;
    st.any[0] = a;
  }
}

// Skinny products with U (n x r, row major) on the float64 matrix cores.  The
// C <= 16 columns sit in the 16 columns of a product (those past C read column
// C - 1 and are dropped).

// W partial: wpart[s][a][c] = sum_{i in split s} Ur[i][a] V[i][c].  A
// workgroup takes 64 columns a of one row split; its four waves take every
// fourth 16 rows of the split and add in LDS.
template <int C>
__global__ __launch_bounds__(PC_TPB) void pc_lt_kernel(const double* __restrict__ Ur, int64_t n, int r,
                                                       const double* __restrict__ V, int64_t rows_per_split,
                                                       double* __restrict__ wpart, const int* __restrict__ gate) {
  NK_PCG_GATE(gate)
  __shared__ double red[4][64 * 16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int a0 = blockIdx.x * 64, c = i < C ? i : C - 1;
  const int64_t i0 = (int64_t)blockIdx.y * rows_per_split;
  const int64_t i1 = i0 + rows_per_split < n ? i0 + rows_per_split : n;
  int a[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) a[b] = a0 + 16 * b + i < r ? a0 + 16 * b + i : r - 1;
  d4 acc[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) acc[b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int64_t q = i0 + 16 * w; q < i1; q += 64) {
    double u[4][4], v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t k = q + 4 * g + t;
      const int64_t kc = k < i1 ? k : i1 - 1;
      v[t] = V[kc * C + c];
      if (k >= i1) v[t] = 0.0;
#pragma unroll
      for (int b = 0; b < 4; ++b) u[b][t] = Ur[kc * r + a[b]];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[b] = mfma64(u[b][t], v[t], acc[b]);
  }
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) red[w][(16 * b + 4 * t + g) * 16 + i] = acc[b][t];
  __syncthreads();
  double* o = wpart + ((int64_t)blockIdx.y * r + a0) * C;
  for (int x = threadIdx.x; x < 64 * C; x += PC_TPB) {
    const int ar = x / C, e = ar * 16 + x - ar * C;
    if (a0 + ar < r) o[x] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
  }
}

// W[a][c] = sum_s wpart[s][a][c]
template <int C>
__global__ __launch_bounds__(64) void pc_w_reduce_kernel(const double* __restrict__ wpart, int S, int r,
                                                         double* __restrict__ W, const int* __restrict__ gate) {
  NK_PCG_GATE(gate)
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= r * C) return;
  double s = 0.0;
#pragma unroll 16
  for (int q = 0; q < S; ++q) s += wpart[(int64_t)q * r * C + e];
  W[e] = s;
}

// Z[i] = (V[i] - sum_a Ur[i][a] W[a]) / lam, PC_ROWS rows per workgroup, 16 per
// wave; partials of v.z per column.
template <int C>
__global__ __launch_bounds__(PC_TPB) void pc_z_kernel(const double* __restrict__ Ur, int64_t n, int r,
                                                      const double* __restrict__ W, const double* __restrict__ V,
                                                      double lam, double* __restrict__ Z,
                                                      double* __restrict__ vz_part, const int* __restrict__ gate) {
  NK_PCG_GATE(gate)
  __shared__ double red[4][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * PC_ROWS + 16 * w;
  const int c = i < C ? i : C - 1;
  const double* pu = Ur + (r0 + i < n ? r0 + i : n - 1) * r + 4 * g;
  const double* pw = W + 4 * g * C + c;
  double vv[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) vv[t] = V[(r0 + 4 * t + g < n ? r0 + 4 * t + g : n - 1) * C + c];
  d4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  int q = 0;
#pragma unroll 2
  for (; q + 32 <= r; q += 32) {
    double u[2][4], b[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      load4(pu + q + 16 * h, u[h]);
#pragma unroll
      for (int t = 0; t < 4; ++t) b[h][t] = pw[(q + 16 * h + t) * C];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[h] = mfma64(u[h][t], b[h][t], acc[h]);
  }
  for (; q < r; q += 16) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bool in = q + 4 * g + t < r;
      acc[0] = mfma64(in ? pu[q + t] : 0.0, in ? pw[(q + t) * C] : 0.0, acc[0]);
    }
  }
  double d = 0.0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double z = (vv[t] - (acc[0][t] + acc[1][t])) / lam;
    const int64_t row = r0 + 4 * t + g;
    if (row < n && i < C) {
      Z[row * C + i] = z;
      d += vv[t] * z;
    }
  }
  d += __shfl_xor(d, 16);
  d += __shfl_xor(d, 32);
  if (g == 0) red[w][i] = d;
  __syncthreads();
  if (threadIdx.x < C)
    vz_part[(int64_t)blockIdx.x * C + threadIdx.x] =
        ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
}

// alpha = gamma / p.q for active columns (0 otherwise); X += alpha P,
// R -= alpha Q; partials of ||r||^2.
template <int C>
__global__ __launch_bounds__(PC_TPB) void pcg_update_kernel(int64_t n, const double* __restrict__ pq_part, int nb,
                                                            PcgState st, int it, const double* __restrict__ P,
                                                            const double* __restrict__ Q, double* __restrict__ X,
                                                            double* __restrict__ R, double* __restrict__ rr_part) {
  const int k = it & 1;
  NK_PCG_GATE(st.any + k)
  __shared__ double red[PC_TPB * C];
  __shared__ double alpha[C];
  pc_colsum<C>(pq_part, nb, red, alpha);
  if (threadIdx.x < C) {
    const int c = threadIdx.x;
    alpha[c] = st.active[16 * k + c] ? st.gamma[16 * k + c] / alpha[c] : 0.0;
  }
  __syncthreads();
  const int64_t e0 = (int64_t)blockIdx.x * PC_ROWS * C, lim = n * C;
  double* prod = red;  // (PC_ROWS * C of it; the column sums below use what follows)
#pragma unroll
  for (int x = threadIdx.x; x < PC_ROWS * C; x += PC_TPB) {
    const int64_t e = e0 + x;
    const double al = alpha[x % C];
    double rv = 0.0;
    if (e < lim) {
      X[e] = fma(al, P[e], X[e]);
      rv = fma(-al, Q[e], R[e]);
      R[e] = rv;
    }
    prod[x] = rv * rv;
  }
  pc_block_sums<C>(prod, red + PC_ROWS * C, rr_part + (int64_t)blockIdx.x * C);
}

// End of iteration `it`: the stopping test on the residuals (rr_part), gamma'
// = r.z (rz_part), beta = gamma' / gamma for columns still active (0
// otherwise), P = Z + beta P; the first workgroup writes the state the next
// iteration reads, and the gate to the host.  it < 0 (after the first
// application of the preconditioner): gamma and P = Z only.
template <int C>
__global__ __launch_bounds__(PC_TPB) void pcg_direction_kernel(int64_t n, const double* __restrict__ rr_part,
                                                               const double* __restrict__ rz_part, int nb,
                                                               PcgState st, int it, double tol,
                                                               const double* __restrict__ Z, double* __restrict__ P,
                                                               int* host_any) {
  const int k = it & 1, kn = it < 0 ? 0 : k ^ 1;
  if (it >= 0 && st.any[k] == 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st.any[kn] = 0;
      if (host_any) __hip_atomic_store(host_any, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  __shared__ double red[PC_TPB * C];
  __shared__ double rr[C], rz[C];
  __shared__ int act[C];
  pc_colsum<C>(rz_part, nb, red, rz);
  if (it >= 0) pc_colsum<C>(rr_part, nb, red, rr);
  if (threadIdx.x < C) {
    const int c = threadIdx.x;
    const double g = rz[c];
    if (it < 0) {
      if (blockIdx.x == 0) st.gamma[c] = g;
      rz[c] = 0.0;
    } else {
      const double old = st.gamma[16 * k + c];
      int a = st.active[16 * k + c];
      if (a) {
        const double rel = sqrt(rr[c]) / st.ynorm[c];
        a = rel <= tol ? 0 : 1;
        if (blockIdx.x == 0) {
          st.relres[c] = rel;
          st.iters[c] = it + 1;
        }
      }
      act[c] = a;
      rz[c] = a ? g / old : 0.0;
      if (blockIdx.x == 0) {
        st.gamma[16 * kn + c] = a ? g : old;
        st.active[16 * kn + c] = a;
      }
    }
  }
  __syncthreads();
  if (it >= 0 && blockIdx.x == 0 && threadIdx.x == 0) {
    int a = 0;
    for (int c = 0; c < C; ++c) a |= act[c];
    st.any[kn] = a;
    if (host_any) __hip_atomic_store(host_any, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  const int64_t e0 = (int64_t)blockIdx.x * PC_ROWS * C, lim = n * C;
#pragma unroll
  for (int x = threadIdx.x; x < PC_ROWS * C; x += PC_TPB) {
    const int64_t e = e0 + x;
    if (e < lim) P[e] = it < 0 ? Z[e] : fma(rz[x % C], P[e], Z[e]);
  }
}

// X[:, c0:c0+C] of the caller's n x ldx output
template <int C>
__global__ __launch_bounds__(PC_TPB) void pcg_store_kernel(int64_t n, const double* __restrict__ Xg,
                                                           double* __restrict__ X, int64_t ldx, int64_t c0) {
  const int64_t e = (int64_t)blockIdx.x * PC_TPB + threadIdx.x;
  if (e >= n * C) return;
  const int64_t i = e / C;
  const int c = (int)(e - i * C);
  X[i * ldx + c0 + c] = Xg[e];
}

// One CG pass over a group of C <= 16 right-hand-side columns.  The host
// enqueues iterations ahead of the device and reads the gate of iteration
// it - 2 (written by its last kernel into pinned host memory, behind an event)
// before enqueueing iteration it, so the device never waits for the host;
// iterations enqueued after every column stopped return at once.
template <int C>
int pcg_group(const PcgArgs& a, int64_t c0, hipStream_t s) {
  const int64_t n = a.n;
  const int nb = (int)((n + PC_ROWS - 1) / PC_ROWS);
  PcgState st{a.gamma, a.ynorm, a.relres, a.active, a.iters, a.any};
  const int lt_splits = a.lt_splits;
  const int64_t lt_rows = (n + lt_splits - 1) / lt_splits;

  auto precond = [&](const double* V, double* Z, double* vz_part, const int* gate) {
    if (a.r > 0) {
      hipLaunchKernelGGL((pc_lt_kernel<C>), dim3((unsigned)((a.r + 63) / 64), (unsigned)lt_splits), dim3(PC_TPB), 0, s,
                         a.Ur, n, a.r, V, lt_rows, a.wpart, gate);
      hipLaunchKernelGGL((pc_w_reduce_kernel<C>), dim3((unsigned)((a.r * C + 63) / 64)), dim3(64), 0, s, a.wpart,
                         lt_splits, a.r, a.W, gate);
    }
    hipLaunchKernelGGL((pc_z_kernel<C>), dim3(nb), dim3(PC_TPB), 0, s, a.Ur, n, a.r, a.W, V, a.lam, Z, vz_part, gate);
  };

  hipLaunchKernelGGL((pcg_init_kernel<C>), dim3(nb), dim3(PC_TPB), 0, s, a.Y, a.ldy, c0, n, a.R, a.X, a.part1);
  hipLaunchKernelGGL((pcg_init_state_kernel<C>), dim3(1), dim3(PC_TPB), 0, s, a.part1, nb, st);
  precond(a.R, a.Z, a.part2, a.any);
  hipLaunchKernelGGL((pcg_direction_kernel<C>), dim3(nb), dim3(PC_TPB), 0, s, n, a.part1, a.part2, nb, st, -1, a.tol,
                     a.Z, a.P, nullptr);
  if (hipGetLastError() != hipSuccess) return -3;

  int rc = 0;
  hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
  for (int e = 0; e < 3 && rc == 0; ++e)
    if (hipEventCreateWithFlags(&ev[e], hipEventDisableTiming) != hipSuccess) rc = -3;
  for (int it = 0; it < a.max_iter && rc == 0; ++it) {
    if (it >= 2) {
      if (hipEventSynchronize(ev[(it - 2) % 3]) != hipSuccess) {
        rc = -3;
        break;
      }
      if (reinterpret_cast<volatile int*>(a.host_any)[(it - 2) % 3] == 0) break;
    }
    const int* gate = a.any + (it & 1);
    if (launch_kmv_c<C>(a.K, n, a.ldk, a.P, a.lam, a.kpart, a.Q, a.part1, gate, s, a.hook)) {
      rc = -3;
      break;
    }
    hipLaunchKernelGGL((pcg_update_kernel<C>), dim3(nb), dim3(PC_TPB), 0, s, n, a.part1, nb, st, it, a.P, a.Q, a.X, a.R,
                       a.part2);
    precond(a.R, a.Z, a.part1, gate);
    hipLaunchKernelGGL((pcg_direction_kernel<C>), dim3(nb), dim3(PC_TPB), 0, s, n, a.part2, a.part1, nb, st, it, a.tol,
                       a.Z, a.P, &a.host_any[it % 3]);
    if (hipEventRecord(ev[it % 3], s) != hipSuccess || hipGetLastError() != hipSuccess) rc = -3;
  }
  for (int e = 0; e < 3; ++e)
    if (ev[e]) (void)hipEventDestroy(ev[e]);
  if (rc) return rc;
  const unsigned gv = (unsigned)((n * C + PC_TPB - 1) / PC_TPB);
  hipLaunchKernelGGL((pcg_store_kernel<C>), dim3(gv), dim3(PC_TPB), 0, s, n, a.X, a.Xout, a.ldx, c0);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_pcg_group(const PcgArgs& a, int64_t c0, int C, hipStream_t s) {
  switch (C) {
    case 1: return pcg_group<1>(a, c0, s);
    case 2: return pcg_group<2>(a, c0, s);
    case 3: return pcg_group<3>(a, c0, s);
    case 4: return pcg_group<4>(a, c0, s);
    case 5: return pcg_group<5>(a, c0, s);
    case 6: return pcg_group<6>(a, c0, s);
    case 7: return pcg_group<7>(a, c0, s);
    case 8: return pcg_group<8>(a, c0, s);
    case 9: return pcg_group<9>(a, c0, s);
    case 10: return pcg_group<10>(a, c0, s);
    case 11: return pcg_group<11>(a, c0, s);
    case 12: return pcg_group<12>(a, c0, s);
    case 13: return pcg_group<13>(a, c0, s);
    case 14: return pcg_group<14>(a, c0, s);
    case 15: return pcg_group<15>(a, c0, s);
    case 16: return pcg_group<16>(a, c0, s);
    default: return -1;
  }
}

int launch_kmv(const float* K, int64_t n, int64_t ldk, const double* P, int C, double lam, double* part, double* Q,
               double* pq_part, hipStream_t s, ProfHook* hook) {
  switch (C) {
#define NK_KMV_CASE(c) \
  case c:              \
    return launch_kmv_c<c>(K, n, ldk, P, lam, part, Q, pq_part, nullptr, s, hook);
    NK_KMV_CASE(1) NK_KMV_CASE(2) NK_KMV_CASE(3) NK_KMV_CASE(4) NK_KMV_CASE(5) NK_KMV_CASE(6) NK_KMV_CASE(7)
    NK_KMV_CASE(8) NK_KMV_CASE(9) NK_KMV_CASE(10) NK_KMV_CASE(11) NK_KMV_CASE(12) NK_KMV_CASE(13)
    NK_KMV_CASE(14) NK_KMV_CASE(15) NK_KMV_CASE(16)
#undef NK_KMV_CASE
    default:
      return -1;
  }
}

// out[0] = mean(diag K)
__global__ __launch_bounds__(PC_TPB) void pc_diag_mean_kernel(const float* __restrict__ K, int64_t n, int64_t ldk,
                                                              double* __restrict__ out) {
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += PC_TPB) s += (double)K[i * ldk + i];
  pc_block_sum_store(s, out);
  if (threadIdx.x == 0) out[0] = out[0] / (double)n;
}

int launch_diag_mean(const float* K, int64_t n, int64_t ldk, double* out, hipStream_t s) {
  hipLaunchKernelGGL(pc_diag_mean_kernel, dim3(1), dim3(PC_TPB), 0, s, K, n, ldk, out);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace nk
