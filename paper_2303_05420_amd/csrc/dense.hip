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
// quantity, rounded once.  Every row x of op(A) and column y of op(B) is split
// into the `bits` leading bits, counted from the largest magnitude in it (top_a,
// top_b), and the rest, x = xh + xl.  A wave's sums of xh yh are then exact in
// float64 (2 bits + log2(terms) <= 53, dn_bits); those of xh yl + xl y are
// 2^-bits of them and carry the rounding errors, about 2^-(52 + bits) of the
// terms' magnitudes in all.  The waves' exact sums meet by TwoSum, the rest is
// added at the end.  Three products for one: the 1000 x 1000 x 12000 product of a
// Nystrom solve takes 738 us.  (Every product's and every addition's error carried on
// the vector unit: 3.8 ms; TwoSum once per 32 plainly summed terms, which loses
// what is below 2^-53 of a larger neighbour: 564.)
// sym: op(B) = op(A)^T; the tiles on and below the diagonal are formed and
// mirrored (a launch of all tiles, half of which return at once, leaves the XCDs
// unevenly loaded: 1222 us for the product above with 32 x 32 tiles, 946 so).

// High word of a number's magnitude: its order, and the exponent above bit 20.
__device__ __forceinline__ unsigned dn_word(double x) {
  return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32) & 0x7fffffffu;
}

// Constant whose addition and subtraction leave the leading `bits` bits of
// numbers up to the one that `top` is the word of (NaN where that is not finite).
__device__ __forceinline__ double dn_splitter(unsigned top, int bits) {
  const unsigned e = (top >> 20) + 53 - (unsigned)bits;
  const unsigned w = (top >> 20) == 0x7ff || e > 0x7fe ? 0x7ff80000u : (e << 20 | 0x80000u);
  return __builtin_bit_cast(double, (unsigned long long)w << 32);
}

template <typename TA, typename TB, typename TO, bool A_T, bool B_T, bool COMP, int MB, int W>
__global__ __launch_bounds__(64 * W, MB == 2 ? (COMP ? 2 : 3) : 1) void dn_gemm_kernel(const TA* __restrict__ A, int64_t lda,
                                                         const TB* __restrict__ B, int64_t ldb, TO* __restrict__ Cm,
                                                         int64_t ldc, int64_t M, int64_t N, int64_t K, double alpha,
                                                         double beta, double shift, int sym, int* __restrict__ info,
                                                         unsigned ntc, const unsigned* __restrict__ top_a,
                                                         const unsigned* __restrict__ top_b, int bits) {
  constexpr int T = 16 * MB, E = T * T;
  extern __shared__ double red[];  // (COMP ? 2 : 1) * W / 2 * E
  unsigned tr = blockIdx.x / ntc, tc = blockIdx.x - tr * ntc;  // tile row and column
  if (sym) {  // (only the tiles on and below the diagonal are launched)
    tr = (unsigned)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
    while (tr * (tr + 1) / 2 > blockIdx.x) --tr;
    while ((tr + 1) * (tr + 2) / 2 <= blockIdx.x) ++tr;
    tc = blockIdx.x - tr * (tr + 1) / 2;
  }
  if (info && blockIdx.x == 0 && threadIdx.x == 0) info[0] = 0;
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  // Where this lane's elements of a chunk are, kept from chunk to chunk (64-bit
  // index products at every load would cost more than the loads).
  struct Place {
    const TA* a[MB][A_T ? 4 : 1];
    const TB* b[MB][B_T ? 1 : 4];
  };
  auto place = [&](int64_t q, Place& p) {
    const int64_t k = 16 * q + 4 * g;
#pragma unroll
    for (int x = 0; x < MB; ++x) {
#pragma unroll
      for (int t = 0; t < (A_T ? 4 : 1); ++t) p.a[x][t] = A_T ? A + (k + t) * lda + ra[x] : A + ra[x] * lda + k;
#pragma unroll
      for (int t = 0; t < (B_T ? 1 : 4); ++t) p.b[x][t] = B_T ? B + cb[x] * ldb + k : B + (k + t) * ldb + cb[x];
    }
  };
  const int64_t step_a = 16 * W * (A_T ? lda : 1), step_b = 16 * W * (B_T ? 1 : ldb);
  auto advance = [&](Place& p, bool on) {
    const int64_t da = on ? step_a : 0, db = on ? step_b : 0;
#pragma unroll
    for (int x = 0; x < MB; ++x) {
#pragma unroll
      for (int t = 0; t < (A_T ? 4 : 1); ++t) p.a[x][t] += da;
#pragma unroll
      for (int t = 0; t < (B_T ? 1 : 4); ++t) p.b[x][t] += db;
    }
  };
  auto fetch = [&](const Place& p, Frag& f) {  // a whole chunk
#pragma unroll
    for (int x = 0; x < MB; ++x) {
      if constexpr (A_T) {
#pragma unroll
        for (int t = 0; t < 4; ++t) f.a[x][t] = *p.a[x][t];
      } else {
        load4(p.a[x][0], f.a[x]);
      }
      if constexpr (B_T) {
        load4(p.b[x][0], f.b[x]);
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) f.b[x][t] = *p.b[x][t];
      }
    }
  };
  // the last chunk, of fewer than 16 (0 past the end)
  const int64_t whole = K / 16;
  auto fetch_rest = [&](Frag& f) {
    const int64_t k = 16 * whole + 4 * g;
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bool in = k + t < K;
        f.a[x][t] = in ? (A_T ? A[(k + t) * lda + ra[x]] : A[ra[x] * lda + k + t]) : (TA)0;
        f.b[x][t] = in ? (B_T ? B[cb[x] * ldb + k + t] : B[(k + t) * ldb + cb[x]]) : (TB)0;
      }
  };
  const bool rest = K % 16 != 0 && whole % W == w;
  // whole chunks w, w + W, ...: two register sets, the next chunk's loads in
  // flight while one is used (past the last: that one again, not used)
  auto walk = [&](auto&& use) {
    if (w < whole) {
      Frag even, odd;
      Place p;
      place(w, p);
      fetch(p, even);
      for (int64_t q = w;;) {
        const bool more = q + W < whole;
        advance(p, more);
        fetch(p, odd);
        use(even);
        if (more) {
          q += 2 * W;
          advance(p, q < whole);
          fetch(p, even);
          use(odd);
        }
        if (!more || q >= whole) break;
      }
    }
    if (rest) {
      Frag f;
      fetch_rest(f);
      use(f);
    }
  };
  double sa[MB], sb[MB];  // COMP: this lane's splitters
  if constexpr (COMP) {
    __shared__ unsigned top[2][T];
    if (tid < 2 * T) top[tid / T][tid % T] = 0;
    __syncthreads();
    unsigned ta[MB], tb[MB];
#pragma unroll
    for (int x = 0; x < MB; ++x) ta[x] = tb[x] = 0;
    if (!top_a || !top_b)
      walk([&](const Frag& f) {
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const unsigned u = dn_word((double)f.a[x][t]), v = dn_word((double)f.b[x][t]);
            ta[x] = u > ta[x] ? u : ta[x];
            tb[x] = v > tb[x] ? v : tb[x];
          }
      });
#pragma unroll
    for (int x = 0; x < MB; ++x) {
      atomicMax(&top[0][16 * x + i], ta[x]);
      atomicMax(&top[1][16 * x + i], tb[x]);
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < MB; ++x) {
      sa[x] = dn_splitter(top_a ? top_a[ra[x]] : top[0][16 * x + i], bits);
      sb[x] = dn_splitter(top_b ? top_b[cb[x]] : top[1][16 * x + i], bits);
    }
  }
  d4 hi[MB][MB], lo[MB][MB];
#pragma unroll
  for (int x = 0; x < MB; ++x)
#pragma unroll
    for (int y = 0; y < MB; ++y) hi[x][y] = lo[x][y] = d4{0.0, 0.0, 0.0, 0.0};
  walk([&](const Frag& f) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      double a[MB], b[MB];
#pragma unroll
      for (int x = 0; x < MB; ++x) {
        a[x] = (double)f.a[x][t];
        b[x] = (double)f.b[x][t];
      }
      if constexpr (COMP) {
        double ah[MB], bh[MB];
#pragma unroll
        for (int x = 0; x < MB; ++x) {
          ah[x] = (a[x] + sa[x]) - sa[x];
          bh[x] = (b[x] + sb[x]) - sb[x];
        }
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
          for (int y = 0; y < MB; ++y) hi[x][y] = mfma64(ah[x], bh[y], hi[x][y]);
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
          for (int y = 0; y < MB; ++y) lo[x][y] = mfma64(ah[x], b[y] - bh[y], lo[x][y]);
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
          for (int y = 0; y < MB; ++y) lo[x][y] = mfma64(a[x] - ah[x], b[y], lo[x][y]);
      } else {
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
          for (int y = 0; y < MB; ++y) hi[x][y] = mfma64(a[x], b[y], hi[x][y]);
      }
    }
  });
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

// Leading bits b for exact sums of `terms` products of b bits each: 2 b +
// log2(terms) <= 53 (20 up to 8192 terms a wave).
static int dn_bits(int64_t terms) {
  int b = 20;
  while (b > 1 && (terms >> (53 - 2 * b)) > 0) --b;
  return b;
}

template <typename TA, typename TB, typename TO, bool A_T, bool B_T, bool COMP, int MB, int W>
static int dn_gemm_launch(const TA* A, int64_t lda, const TB* B, int64_t ldb, TO* C, int64_t ldc, int64_t M, int64_t N,
                          int64_t K, double alpha, double beta, hipStream_t s, double shift, bool sym, int* info,
                          const unsigned* top_a, const unsigned* top_b) {
  static std::atomic<size_t> seen[kMaxDevices];
  constexpr int T = 16 * MB;
  const size_t lds = (size_t)(COMP ? 2 : 1) * W / 2 * T * T * sizeof(double);
  const auto kernel = dn_gemm_kernel<TA, TB, TO, A_T, B_T, COMP, MB, W>;
  if (allow_dyn_lds((const void*)kernel, lds, seen)) return -3;
  const int64_t mt = (M + T - 1) / T, nt = (N + T - 1) / T;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(sym ? mt * (mt + 1) / 2 : mt * nt)), dim3(64 * W), lds, s, A, lda, B, ldb,
                     C, ldc, M, N, K, alpha, beta, shift, sym ? 1 : 0, info, (unsigned)nt, top_a, top_b,
                     dn_bits((K / 16 + W) / W * 16));
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Tile by size: 16 x 16 with up to 16 waves on a long sum, until 32 x 32 tiles
// (half the operand traffic and conversions) reach every CU.
template <typename TA, typename TB, typename TO, bool A_T, bool B_T, bool COMP>
static int dn_gemm_t(const TA* A, int64_t lda, const TB* B, int64_t ldb, TO* C, int64_t ldc, int64_t M, int64_t N,
                     int64_t K, double alpha, double beta, hipStream_t s, double shift = 0.0, bool sym = false,
                     int* info = nullptr, const unsigned* top_a = nullptr, const unsigned* top_b = nullptr) {
  if (M <= 0 || N <= 0) return 0;
  const int64_t m = (M + 31) / 32, n = (N + 31) / 32, h = (M + 15) / 16;
  const auto go = [&](auto launch) {
    return launch(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s, shift, sym, info, top_a, top_b);
  };
  if constexpr (COMP && (A_T || B_T)) {  // (the forms that have symmetric results)
    // Three products for one make the last round dear: 32 x 32 tiles of a
    // symmetric result only from four a CU on.  1000 x 1000 x 12000, 528 of them
    // 946 us, 2016 of 16 x 16 with four waves 766, with eight 738.
    if (sym && h * (h + 1) / 2 >= 512 && m * (m + 1) / 2 < 1024)
      return go(dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 1, 8>);
  }
  if (N > 16 && (sym ? m * (m + 1) / 2 : m * n) >= 256) return go(dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 2, 4>);
  return K > 256 ? go(dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 1, 16>)
                 : go(dn_gemm_launch<TA, TB, TO, A_T, B_T, COMP, 1, 4>);
}

// top[c] = largest word of column c of A (n x r, lda), zero before.
__global__ __launch_bounds__(256) void dn_column_top_kernel(const float* __restrict__ A, int64_t lda, int64_t n,
                                                            int64_t r, int64_t rows, unsigned* __restrict__ top) {
  __shared__ unsigned part[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t c = (int64_t)blockIdx.x * 64 + lane, i0 = (int64_t)blockIdx.y * rows;
  const int64_t i1 = i0 + rows < n ? i0 + rows : n;
  const float* p = A + (c < r ? c : r - 1);
  unsigned m = 0;
#pragma unroll 8
  for (int64_t i = i0 + w; i < i1; i += 4) {
    const unsigned u = __builtin_bit_cast(unsigned, p[i * lda]) & 0x7fffffffu;
    m = u > m ? u : m;
  }
  part[w][lane] = m;
  __syncthreads();
  if (w != 0 || c >= r) return;
  for (int k = 1; k < 4; ++k) m = part[k][lane] > m ? part[k][lane] : m;
  atomicMax(&top[c], dn_word((double)__builtin_bit_cast(float, m)));
}

int dn_column_top(const float* A, int64_t lda, int64_t n, int64_t r, unsigned* top, hipStream_t s) {
  if (launch_zero_f64(reinterpret_cast<double*>(top), (r + 1) / 2, s)) return -3;
  const int64_t cb = (r + 63) / 64;
  int64_t parts = (1024 + cb - 1) / cb;
  if (parts > (n + 63) / 64) parts = (n + 63) / 64;
  const int64_t rows = (n + parts - 1) / parts;
  hipLaunchKernelGGL(dn_column_top_kernel, dim3((unsigned)cb, (unsigned)parts), dim3(256), 0, s, A, lda, n, r, rows,
                     top);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int dn_gemm_ff(const float* A, int64_t lda, bool a_t, const float* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
               int64_t N, int64_t K, double alpha, double beta, bool comp, hipStream_t s, const unsigned* top_a, const unsigned* top_b) {
  if (!a_t || !comp) return -1;  // (only the compensated A^T B is used)
  const bool sym = A == B && lda == ldb && M == N && beta == 0.0;
  return dn_gemm_t<float, float, double, true, false, true>(A, lda, B, ldb, C, ldc, M, N, K, alpha, beta, s, 0.0, sym,
                                                            nullptr, top_a, top_b);
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
  const double v = (double)S[i * lds + j];
  D[e] = i == j ? chol_diagonal(v + shift) : v;
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
  if (i < n) D[i * n + i] = chol_diagonal(D[i * n + i] + shift);
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
