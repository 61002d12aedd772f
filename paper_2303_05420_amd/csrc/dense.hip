// Dense float64 building blocks of the approximate kernel-regression solvers
// (Sec. 2, "Approximations to the linear system"; sequenced by the host API
// entry points nk_krr_nystrom, nk_krr_sor, nk_krr_block_diag, nk_krr_bcm): a tiled
// GEMM with float32 or float64 operands and float64 accumulation (optionally
// compensated), symmetric-matrix loads with a diagonal shift, identity
// fills, row updates and casts.
#include "mfma64.h"

namespace nk {

// C (M x N, TO, ldc) = beta C + alpha op(A) op(B), plus shift I.
//   op(A) = A (M x K, lda) or, with A_T, A^T where A is K x M (lda); op(B) = B
//   (K x N, ldb) or, with B_T, B^T where B is N x K (ldb); all row-major.
// A workgroup owns a square tile of MB x MB blocks of 16 x 16 on the float64
// matrix cores; its W waves take every W-th chunk of 16 k each and meet in
// LDS at the end, in a fixed order, so a tile's sum is spread over a CU
// however few tiles there are.  Operands come straight from the caches (a
// lane's four consecutive k of a row, or 16 lanes' consecutive columns), the
// next chunk's while the current one runs.  Bound: the float64 pipes, shared
// by the products (4 MB^2 of 64 cycles a chunk), the operands' conversions and
// COMP's sums; reading the operands from a cached 256 rows instead changes
// nothing.
// COMP: for sums whose result is later subtracted from a nearly equal
// quantity.  Two chunks start from zero and their sum is added to the running
// one with TwoSum, the rounding errors carried and added at the end: what is
// left is the rounding inside 32 terms of a sum of K, and one rounding of the
// result.  (A chain of compensated single products on the vector unit, 4
// outputs per thread: 3.8 ms for the 1000 x 1000 x 12000 product of a
// Nystrom solve, now 0.57.)
// sym: op(B) = op(A)^T; the tiles on and below the diagonal are formed and
// mirrored.
template <typename TA, typename TB, typename TO, bool A_T, bool B_T, bool COMP, int MB, int W>
__global__ __launch_bounds__(64 * W, MB == 2 ? 3 : 1) void dn_gemm_kernel(const TA* __restrict__ A, int64_t lda,
                                                         const TB* __restrict__ B, int64_t ldb, TO* __restrict__ Cm,
                                                         int64_t ldc, int64_t M, int64_t N, int64_t K, double alpha,
                                                         double beta, double shift, int sym, int* __restrict__ info,
                                                         unsigned ntc) {
  constexpr int T = 16 * MB, E = T * T;
  extern __shared__ double red[];  // (COMP ? 2 : 1) * W / 2 * E
  const unsigned tr = blockIdx.x / ntc, tc = blockIdx.x - tr * ntc;  // tile row and column
  if (info && blockIdx.x == 0 && threadIdx.x == 0) info[0] = 0;
  if (sym && tc > tr) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int64_t r0 = (int64_t)tr * T, c0 = (int64_t)tc * T;
  int64_t ra[MB], cb[MB];  // this lane's rows of op(A) and columns of op(B) (past the end: the last one, not stored)
#pragma unroll
  for (int x = 0; x < MB; ++x) {
    ra[x] = r0 + 16 * x + i < M ? r0 + 16 * x + i : M - 1;
    cb[x] = c0 + 16 * x + i < N ? c0 + 16 * x + i : N - 1;
  }
  struct Frag {
    TA a[MB][4];
    TB b[MB][4];
  };
  auto fetch = [&](int64_t q, Frag& f) {  // chunk q, a whole one
    const int64_t k = 16 * q + 4 * g;
#pragma unroll
    for (int x = 0; x < MB; ++x) {
      if constexpr (A_T) {
#pragma unroll
        for (int t = 0; t < 4; ++t) f.a[x][t] = A[(k + t) * lda + ra[x]];
      } else {
        load4(A + ra[x] * lda + k, f.a[x]);
      }
      if constexpr (B_T) {
        load4(B + cb[x] * ldb + k, f.b[x]);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) f.b[x][t] = B[(k + t) * ldb + cb[x]];
      }
    }
  };
  d4 hi[MB][MB], lo[MB][MB];
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int y = 0; y < MB; ++y) hi[x][y] = lo[x][y] = d4{0.0, 0.0, 0.0, 0.0};
  auto multiply = [&](const Frag& f, d4 (&p)[MB][MB]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < MB; ++y) p[x][y] = mfma64((double)f.a[x][t], (double)f.b[y][t], p[x][y]);
  };
  d4 p[MB][MB];  // COMP: the running chunk pair
  auto start = [&]() {
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
      for (int y = 0; y < MB; ++y) p[x][y] = d4{0.0, 0.0, 0.0, 0.0};
  };
  auto add = [&]() {
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
      for (int y = 0; y < MB; ++y) {
        const d4 s = hi[x][y] + p[x][y];
        const d4 bb = s - hi[x][y];
        lo[x][y] += (hi[x][y] - (s - bb)) + (p[x][y] - bb);
        hi[x][y] = s;
      }
  };
  // whole chunks w, w + W, ...: two register sets, the next chunk's loads in
  // flight while one multiplies (past the last: that one again, not used)
  const int64_t whole = K / 16;
  if (w < whole) {
    Frag even, odd;
    fetch(w, even);
    for (int64_t q = w;;) {
      const bool more = q + W < whole;
      fetch(more ? q + W : q, odd);
      if (COMP) start();
      multiply(even, COMP ? p : hi);
      if (more) {
        q += 2 * W;
        fetch(q < whole ? q : q - W, even);
        multiply(odd, COMP ? p : hi);
      }
      if (COMP) add();
      if (!more || q >= whole) break;
    }
  }
  if (K % 16 != 0 && whole % W == w) {
    Frag f;
    const int64_t k = 16 * whole + 4 * g;
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bool in = k + t < K;
        f.a[x][t] = in ? (A_T ? A[(k + t) * lda + ra[x]] : A[ra[x] * lda + k + t]) : (TA)0;
        f.b[x][t] = in ? (B_T ? B[cb[x] * ldb + k + t] : B[(k + t) * ldb + cb[x]]) : (TB)0;
      }
    if (COMP) start();
    multiply(f, COMP ? p : hi);
    if (COMP) add();
  }
  // the upper half of the waves into the lower one, until one is left
#pragma unroll 1
  for (int h = W / 2; h >= 1; h >>= 1) {
    double* mine = red + (size_t)(w % h) * E * (COMP ? 2 : 1);
    if (w >= h && w < 2 * h) {
#pragma unroll
      for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < MB; ++y)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int e = ((x * MB + y) * 4 + v) * 64 + lane;
            mine[e] = hi[x][y][v];
            if (COMP) mine[E + e] = lo[x][y][v];
          }
    }
    __syncthreads();
    if (w < h) {
#pragma unroll
      for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int y = 0; y < MB; ++y)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int e = ((x * MB + y) * 4 + v) * 64 + lane;
            const double o = mine[e];
            if (COMP) {
              const double s = hi[x][y][v] + o, bb = s - hi[x][y][v];
              lo[x][y][v] += (hi[x][y][v] - (s - bb)) + (o - bb) + mine[E + e];
              hi[x][y][v] = s;
            } else {
              hi[x][y][v] += o;
            }
          }
    }
    __syncthreads();
  }
  if (w != 0) return;
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int y = 0; y < MB; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + 16 * x + 4 * v + g, c = c0 + 16 * y + i;
        if (r >= M || c >= N || (sym && c > r)) continue;
        double s = hi[x][y][v], l = lo[x][y][v];
        if (COMP && r == c && shift != 0.0) {
          const double u = s + shift, bb = u - s;
          l += (s - (u - bb)) + (shift - bb);
          s = u;
        }
        const double val = alpha * (s + l);
        TO* o = Cm + r * ldc + c;
        const double out = beta == 0.0 ? val : __builtin_fma(beta, (double)*o, val);
        *o = (TO)out;
        if (sym && c < r) Cm[c * ldc + r] = (TO)out;
      }
}

template <typename TA, typename TB, typename TO, bool A_T, bool B_T, bool COMP, int MB, int W>
static int dn_gemm_launch(const TA* A, int64_t lda, const TB* B, int64_t ldb, TO* C, int64_t ldc, int64_t M, int64_t N,
                          int64_t K, double alpha, double beta, hipStream_t s, double shift, bool sym, int* info) {
  static std::atomic<size_t> seen[kMaxDevices];
  constexpr int T = 16 * MB;
  const size_t lds = (size_t)(COMP ? 2 : 1) * W / 2 * T * T * sizeof(double);
  const auto kernel = dn_gemm_kernel<TA, TB, TO, A_T, B_T, COMP, MB, W>;
  if (allow_dyn_lds((const void*)kernel, lds, seen)) return -3;
  const int64_t mt = (M + T - 1) / T, nt = (N + T - 1) / T;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(mt * nt)), dim3(64 * W), lds, s, A, lda, B, ldb, C, ldc, M, N, K, alpha,
                     beta, shift, sym ? 1 : 0, info, (unsigned)nt);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Tile by size: 16 x 16 with up to 16 waves on a long sum, until 32 x 32 tiles
// (half the operand traffic and conversions) reach every CU.
template <typename TA, typename TB, typename TO, bool A_T, bool B_T, bool COMP>
static int dn_gemm_t(const TA* A, int64_t lda, const TB* B, int64_t ldb, TO* C, int64_t ldc, int64_t M, int64_t N,
                     int64_t K, double alpha, double beta, hipStream_t s, double shift = 0.0, bool sym = false,
                     int* info = nullptr) {
  if (M <= 0 || N <= 0) return 0;
  const int64_t m = (M + 31) / 32, n = (N + 31) / 32;
  if (N > 16 && (sym ? m * (m + 1) / 2 : m * n) >= 256)
    return dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 2, 4>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s, shift, sym,
                                                            info);
  return K > 256 ? dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 1, 16>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s,
                                                                     shift, sym, info)
                 : dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 1, 4>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s,
                                                                    shift, sym, info);
}

int dn_gemm_ff(const float* A, int64_t lda, bool a_t, const float* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
               int64_t N, int64_t K, double alpha, double beta, bool comp, hipStream_t s) {
  if (!a_t || !comp) return -1;  // (only the compensated A^T B is used)
  const bool sym = A == B && lda == ldb && M == N && beta == 0.0;
  return dn_gemm_t<float, float, double, true, false, true>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s, 0.0, sym);
}

int dn_gemm_fd(const float* A, int64_t lda, bool a_t, const double* B, int64_t ldb, double* C, int64_t ldc,
               int64_t M, int64_t N, int64_t K, double alpha, double beta, bool comp, hipStream_t s) {
  if (a_t) {
    if (comp) return -1;
    return dn_gemm_t<float, double, double, true, false, false>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s);
  }
  return comp ? dn_gemm_t<float, double, double, false, false, true>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s)
              : dn_gemm_t<float, double, double, false, false, false>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s);
}

int dn_gemm_dd(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
               int64_t N, int64_t K, double alpha, double beta, hipStream_t s) {
  return dn_gemm_t<double, double, double, false, false, false>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s);
}

int dn_gemm_fdf(const float* A, int64_t lda, const double* B, int64_t ldb, float* C, int64_t ldc, int64_t M,
                int64_t N, int64_t K, hipStream_t s) {
  return dn_gemm_t<float, double, float, false, false, false>(A, lda, B, ldb, C, ldc, M, N, K, 1.0, 0.0, s);
}

int dn_ltl(const double* L, int64_t n, int64_t r, double lam, double* M, int* info, hipStream_t s) {
  return dn_gemm_t<double, double, double, false, true, true>(L, n, L, n, M, r, r, r, n, 1.0, 0.0, s, lam, true, info);
}

// D (n x n, double, dense) = S (float, lds) + shift I; clears info[0] when given.
__global__ __launch_bounds__(256) void dn_load_shift_kernel(const float* __restrict__ S, int64_t lds, int64_t n,
                                                            double shift, double* __restrict__ D,
                                                            int* __restrict__ info) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (info && e == 0) info[0] = 0;
  if (e >= n * n) return;
  const int64_t i = e / n, j = e - i * n;
  D[e] = (double)S[i * lds + j] + (i == j ? shift : 0.0);
}

int dn_load_shift(const float* S, int64_t lds, int64_t n, double shift, double* D, int* info, hipStream_t s) {
  hipLaunchKernelGGL(dn_load_shift_kernel, dim3((unsigned)((n * n + 255) / 256)), dim3(256), 0, s, S, lds, n, shift,
                     D, info);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// D (n x n double) += shift I and (optionally) clears info[0]
__global__ __launch_bounds__(256) void dn_shift_kernel(double* __restrict__ D, int64_t n, double shift,
                                                       int* __restrict__ info) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (info && i == 0) info[0] = 0;
  if (i < n) D[i * n + i] += shift;
}

int dn_shift(double* D, int64_t n, double shift, int* info, hipStream_t s) {
  hipLaunchKernelGGL(dn_shift_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, D, n, shift, info);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// I (n x n double) = identity
__global__ __launch_bounds__(256) void dn_identity_kernel(double* __restrict__ I, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * n) return;
  I[e] = (e / n == e % n) ? 1.0 : 0.0;
}

int dn_identity(double* I, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(dn_identity_kernel, dim3((unsigned)((n * n + 255) / 256)), dim3(256), 0, s, I, n);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// out (rows x cols double, ldo) = in (float, ldi), transposed when trans
__global__ __launch_bounds__(256) void dn_copy_f_kernel(const float* __restrict__ in, int64_t ldi, int64_t rows,
                                                        int64_t cols, bool trans, double* __restrict__ out,
                                                        int64_t ldo) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= rows * cols) return;
  const int64_t i = e / cols, j = e - i * cols;
  out[i * ldo + j] = trans ? (double)in[j * ldi + i] : (double)in[i * ldi + j];
}

int dn_copy_f(const float* in, int64_t ldi, int64_t rows, int64_t cols, bool trans, double* out, int64_t ldo,
              hipStream_t s) {
  if (rows * cols <= 0) return 0;
  hipLaunchKernelGGL(dn_copy_f_kernel, dim3((unsigned)((rows * cols + 255) / 256)), dim3(256), 0, s, in, ldi, rows,
                     cols, trans, out, ldo);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// X (n x c double) = (Yf - X) * scale, Yf float (ldy)
__global__ __launch_bounds__(256) void dn_residual_scale_kernel(const float* __restrict__ Y, int64_t ldy, int64_t n,
                                                                int64_t c, double scale, double* __restrict__ X) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n * c) return;
  const int64_t i = e / c, j = e - i * c;
  X[e] = ((double)Y[i * ldy + j] - X[e]) * scale;
}

int dn_residual_scale(const float* Y, int64_t ldy, int64_t n, int64_t c, double scale, double* X, hipStream_t s) {
  hipLaunchKernelGGL(dn_residual_scale_kernel, dim3((unsigned)((n * c + 255) / 256)), dim3(256), 0, s, Y, ldy, n, c,
                     scale, X);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// out (float, ldo) = in (double, rows x cols dense)
__global__ __launch_bounds__(256) void dn_cast_kernel(const double* __restrict__ in, int64_t rows, int64_t cols,
                                                      float* __restrict__ out, int64_t ldo) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= rows * cols) return;
  const int64_t i = e / cols, j = e - i * cols;
  out[i * ldo + j] = (float)in[e];
}

int dn_cast(const double* in, int64_t rows, int64_t cols, float* out, int64_t ldo, hipStream_t s) {
  if (rows * cols <= 0) return 0;
  hipLaunchKernelGGL(dn_cast_kernel, dim3((unsigned)((rows * cols + 255) / 256)), dim3(256), 0, s, in, rows, cols,
                     out, ldo);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// D = alpha D + beta E elementwise over n doubles (alpha = 0: D is not read)
__global__ __launch_bounds__(256) void dn_axpby_kernel(double* __restrict__ D, const double* __restrict__ E,
                                                       int64_t n, double alpha, double beta) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  D[e] = alpha == 0.0 ? beta * E[e] : __builtin_fma(alpha, D[e], beta * E[e]);
}

int dn_axpby(double* D, const double* E, int64_t n, double alpha, double beta, hipStream_t s) {
  hipLaunchKernelGGL(dn_axpby_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, D, E, n, alpha, beta);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace nk
