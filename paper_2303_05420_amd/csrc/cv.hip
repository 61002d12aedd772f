// CNN-VEC NNGP (App. "Neural Kernel Architecture", CNN-VEC listing: `depth`
// blocks of [3x3 SAME conv, ReLU] at full resolution, Flatten, Dense).
//
// The flatten readout averages the covariance of each pixel of x with the
// same pixel of x', and a conv maps entry (i, j) to (i + d, j + d): so only
// the displacement-0 entries (i, i) are ever needed, one h x w map per pair
// and layer instead of the (h w)^2 of a pooled network.  That map is the
// k = (0, 0) tile of the sheared layout of the Myrtle stage kernel (lane =
// column, register = row, no seam): every pair runs in one N-lane segment
// and carries its tile through all layers in registers.
//
// Tables (cv_prepare_kernel, float64 inside): per image, layer and pixel,
//   alpha = q^{-1/2},  beta = (kappa q / 2)^{1/2},
// q the pre-activation variance of the image at that ReLU (its own
// displacement-0 recursion, where the ReLU map of (q, q, q) is q / 2), kappa
// the scale that multiplies the layer's output downstream: sigma_w2 / 9 of
// the next conv, sigma_w2 / (h w) of the readout after the last layer.  The
// seed's sigma_w2 / (9 C) rides on the second image's pixels.
#include "nk_tile.h"

namespace nk {

// One image per workgroup (the images of x1, then those of x2), one thread per
// pixel (N * N threads).
__global__ void cv_prepare_kernel(const float* __restrict__ x1, int64_t n1, const float* __restrict__ x2, int N, int C,
                                  int D, double sw2, double sb2, float2* __restrict__ tab1,
                                  float2* __restrict__ tab2) {
  extern __shared__ double cv_map[];  // N * N doubles
  double* S = cv_map;
  const int px = threadIdx.x;
  const int iy = px / N, ix = px - iy * N;
  const bool second = blockIdx.x >= n1;
  const int64_t img = second ? blockIdx.x - n1 : blockIdx.x;
  const float* xi = (second ? x2 : x1) + (img * N * N + px) * C;
  double s = 0.0;
  for (int c = 0; c < C; ++c) s += (double)xi[c] * (double)xi[c];
  S[px] = s / C;
  __syncthreads();
  float2* t = (second ? tab2 : tab1) + img * (int64_t)D * N * N;
  for (int l = 0; l < D; ++l) {
    double b = 0.0;
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        const int y = iy + dy, xx = ix + dx;
        if (y >= 0 && y < N && xx >= 0 && xx < N) b += S[y * N + xx];
      }
    const double q = sw2 / 9.0 * b + sb2;
    const double kappa = l + 1 < D ? sw2 / 9.0 : sw2 / (double)(N * N);
    t[(int64_t)l * N * N + px] = make_float2((float)(1.0 / sqrt(q)), (float)sqrt(kappa * q * 0.5));
    __syncthreads();
    S[px] = 0.5 * q;
    __syncthreads();
  }
}

struct CvArgs {
  const float* x1;
  const float* x2;
  int64_t n1, n2;
  int sym, T, C, D;
  const float2* tab1;
  const float2* tab2;
  float* K;
  int64_t ldk;
  float sb2, seed_scale;
  int64_t nb1, nb2, nblocks;  // 4 x 4 pair blocks per side, and in the pass
};

// Workgroup shape.  A workgroup computes a block of 4 x 4 pairs (images
// 4 bi + 0..3 of x1 against 4 bj + 0..3 of x2), one N-lane segment per pair,
// so that the tables of 8 images serve 16 pairs.  Each layer's tables of the
// 8 images sit in LDS (8 N^2 float2: 16 KiB at N = 16); the next layer's are
// fetched into registers while the current layer is computed, and written to
// LDS between two barriers.  (N = 32 has a kernel of its own below.)

// hsum3 plus b: the copy that starts the sum becomes an addition.
__device__ __forceinline__ float hsum3b(float x, float b, float mL, float mR) {
  float h;
  asm("v_add_f32 %0, %1, %4\n\t"
      "s_nop 1\n\t"
      "v_fmac_f32_dpp %0, %1, %2 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
      "v_fmac_f32_dpp %0, %1, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
      : "=&v"(h)
      : "v"(x), "v"(mL), "v"(mR), "v"(b));
  return h;
}

template <int N>
struct CvB {
  static constexpr int PAIRS = 16;
  static constexpr int THREADS = PAIRS * N < 64 ? 64 : PAIRS * N;
  static constexpr int NN = N * N;
  static constexpr size_t LDS = (size_t)8 * NN * sizeof(float2);
  static constexpr int RH = N / 2;  // row before which the next layer's tables are requested
};

// One [3x3 conv, ReLU] layer of a displacement-0 tile (no seam: the
// vertical links are all present), with the forward NNGP's degree-3 fit of
// the map.  The next layer's table float4s of this
// thread (src + m * TPS, m < NV) are requested before row RH, so that the
// registers they land in are live for the rest of the layer only.
template <int N, bool SIGNED, bool BIAS, int RH, int NV, int TPS, bool FULL>
__device__ __forceinline__ void cv_layer(float (&A)[N], const float2* __restrict__ c1,
                                         const float2* __restrict__ c2, float mL, float mR, float sb2,
                                         const float4* __restrict__ src, int sj, int half, float (&pf)[NV][4]) {
  // BIAS: a third of it rides in each row's horizontal sum (interior rows take
  // three of those)
  const float b3 = BIAS ? sb2 * (1.0f / 3.0f) : 0.f;
  auto hsum = [&](float x) { return BIAS ? hsum3b(x, b3, mL, mR) : hsum3(x, mL, mR); };
  float hm = b3;
  float h0 = hsum(A[0]);
#pragma unroll
  for (int r = 0; r < N; ++r) {
    if (r == RH) {
#pragma unroll
      for (int m = 0; m < NV; ++m)
        if (FULL || sj + m * TPS < half) {
          const float4 v = src[m * TPS];
          pf[m][0] = v.x;
          pf[m][1] = v.y;
          pf[m][2] = v.z;
          pf[m][3] = v.w;
        }
    }
    float hp = b3;
    if (r + 1 < N) hp = hsum(A[r + 1]);
    float v = h0;
    if (r > 0 || BIAS) v += hm;
    if (r + 1 < N || BIAS) v += hp;
    const float2 ta = c1[r * N];
    const float2 tb = c2[r * N];
    const float rr = ta.x * tb.x;
    const float J = SIGNED ? j1_signed_vr3(v, rr) : j1_nonneg3(v * rr);
    A[r] = (ta.y * tb.y) * J;
    hm = h0;
    h0 = hp;
  }
}

// Readout of a pair: the tile's sum (its scale rides on the last layer's tables).
template <int N>
__device__ __forceinline__ void cv_readout(const CvArgs& a, const float (&A)[N], int ix, int64_t ia, int64_t ib,
                                           bool valid) {
  float t[N];
#pragma unroll
  for (int r = 0; r < N; ++r) t[r] = A[r];
#pragma unroll
  for (int w = N / 2; w >= 1; w >>= 1) {
#pragma unroll
    for (int r = 0; r < w; ++r) t[r] = t[r] + t[r + w];
  }
  double sum = (double)t[0];
#pragma unroll
  for (int off = N / 2; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, N);
  if (ix == 0 && valid) {
    const float kv = (float)(sum + (double)a.sb2);
    a.K[ia * a.ldk + ib] = kv;
    if (a.sym && ia != ib) a.K[ib * a.ldk + ia] = kv;
  }
}

// Images of 32 x 32: the same 4 x 4 pair block per workgroup (8 waves, two
// workgroups per CU), with the tables in pieces of 8 rows of the 8 images (16
// KiB), a ring of four in LDS, and two more on their way in registers.  So
// the kernel never stops to restage: a step of 8 rows is one barrier, the store of the next piece and the
// request of the third one after it, 16 registers instead of the 32 that a
// layer's tables take, and those 16 go to the row pairs of the vertical sums
// (rows r, r + 1 share h(r) + h(r + 1)).  The kernel is bound by issue
// (VALU busy 93 %); what it saves is instructions: 15 per entry and layer
// (horizontal sum 3 with the bias riding in it, vertical 1.5, map 10) where a
// layer at a time took 18.5 with the copies of the tile around its branch on
// the first layer.  CV8, 1000 x 1030 pairs: 4515 us a call with a layer
// at a time, 4270-4325 so on the same card (both with the tables' 60 to 120 us;
// 4.3 to 4.7 ms from card to card).
constexpr int CV_ROWS = 8, CV_PIECE = 8 * CV_ROWS * 32;  // float2 per piece

struct Cv32 {
  float2* lds;         // [4][8 images][8 rows][32 columns]
  const float4* g[2];  // this thread's float4 of piece 0 of its x1 and its x2 image
  float4* put[2];      // its place in LDS (slot 0)
  int o1, o2;          // this pair's images in a slot, at column ix
  int t, last;         // piece in use, last piece
  int cur;             // float2 offset of the slot in use
  float mL, mR, b3;
};

// Start of the step on piece c.t: R holds piece t + 1 and receives piece t + 3
// (past the last one: that one again, in bounds and not used).
__device__ __forceinline__ void cv32_step(Cv32& c, float (&R)[2][4]) {
  __syncthreads();
  const int nxt = ((c.t + 1) & 3) * CV_PIECE;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    c.put[m][nxt / 2] = make_float4(R[m][0], R[m][1], R[m][2], R[m][3]);
    const int p = c.t + 3 < c.last ? c.t + 3 : c.last;
    const float4 v = c.g[m][p * (CV_PIECE / 16)];
    R[m][0] = v.x;
    R[m][1] = v.y;
    R[m][2] = v.z;
    R[m][3] = v.w;
  }
}

// One [3x3 conv, ReLU] layer of a displacement-0 tile, in place; on entry
// `odd` holds the layer's second piece and `even` its third.
template <bool SIGNED, bool BIAS>
__device__ __forceinline__ void cv32_layer(float (&A)[32], Cv32& c, float (&even)[2][4], float (&odd)[2][4]) {
  auto hsum = [&](float x) { return BIAS ? hsum3b(x, c.b3, c.mL, c.mR) : hsum3(x, c.mL, c.mR); };
  float hm = c.b3, h0 = hsum(A[0]), h1 = hsum(A[1]);
#pragma unroll
  for (int r = 0; r < 32; r += 2) {
    if (r % CV_ROWS == 0) {
      if ((r / CV_ROWS) & 1)
        cv32_step(c, even);
      else
        cv32_step(c, odd);
    }
    const float h2 = r + 2 < 32 ? hsum(A[r + 2]) : c.b3;
    const float h3 = r + 3 < 32 ? hsum(A[r + 3]) : 0.f;
    const float p = h0 + h1;
    const float v0 = r > 0 || BIAS ? p + hm : p, v1 = r + 2 < 32 || BIAS ? p + h2 : p;
    const float2* t1 = c.lds + c.cur + c.o1 + (r % CV_ROWS) * 32;
    const float2* t2 = c.lds + c.cur + c.o2 + (r % CV_ROWS) * 32;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float2 ta = t1[32 * k], tb = t2[32 * k];
      const float v = k == 0 ? v0 : v1, rr = ta.x * tb.x;
      const float J = SIGNED ? j1_signed_vr3(v, rr) : j1_nonneg3(v * rr);
      A[r + k] = (ta.y * tb.y) * J;
    }
    hm = h1;
    h0 = h2;
    h1 = h3;
    if (r % CV_ROWS == CV_ROWS - 2) {
      ++c.t;
      c.cur = (c.t & 3) * CV_PIECE;
    }
  }
}

template <int C, bool BIAS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void cv32_block_kernel(const CvArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, q = tid >> 5, ix = tid & 31;
  const int qa = q >> 2, qb = q & 3;
  int64_t bi, bj;
  pair_of(xcd_logical_block(), a.nb1, a.nb2, a.sym, a.T, &bi, &bj);
  const int64_t ia = bi * 4 + qa, ib = bj * 4 + qb;
  const bool valid = ia < a.n1 && ib < a.n2 && !(a.sym && bi == bj && qa > qb);
  Cv32 c;
  c.lds = reinterpret_cast<float2*>(smem);
  {
    // staging: 128 threads per image, one of x1 and one of x2 each
    const int s = tid >> 7, j = tid & 127;
    const int64_t m1 = bi * 4 + s < a.n1 ? bi * 4 + s : a.n1 - 1, m2 = bj * 4 + s < a.n2 ? bj * 4 + s : a.n2 - 1;
    c.g[0] = reinterpret_cast<const float4*>(a.tab1) + m1 * (int64_t)a.D * 512 + j;
    c.g[1] = reinterpret_cast<const float4*>(a.tab2) + m2 * (int64_t)a.D * 512 + j;
    c.put[0] = reinterpret_cast<float4*>(smem) + s * 128 + j;
    c.put[1] = c.put[0] + 512;
  }
  c.o1 = qa * (CV_ROWS * 32) + ix;
  c.o2 = (4 + qb) * (CV_ROWS * 32) + ix;
  c.t = 0;
  c.last = 4 * a.D - 1;
  c.cur = 0;
  c.mL = ix >= 1 ? 1.f : 0.f;
  c.mR = ix + 1 < 32 ? 1.f : 0.f;
  c.b3 = BIAS ? a.sb2 * (1.0f / 3.0f) : 0.f;
  float even[2][4], odd[2][4];
  {
    float4 z[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const float4 v0 = c.g[m][0], v1 = c.g[m][CV_PIECE / 16], v2 = c.g[m][2 * (CV_PIECE / 16)];
      z[m] = v0;
      odd[m][0] = v1.x;
      odd[m][1] = v1.y;
      odd[m][2] = v1.z;
      odd[m][3] = v1.w;
      even[m][0] = v2.x;
      even[m][1] = v2.y;
      even[m][2] = v2.z;
      even[m][3] = v2.w;
    }
    c.put[0][0] = z[0];
    c.put[1][0] = z[1];
  }
  // seed: the pixels of 4 rows are requested together, then combined
  const float* p1 = a.x1 + ((ia < a.n1 ? ia : a.n1 - 1) * 1024 + ix) * C;
  const float* p2 = a.x2 + ((ib < a.n2 ? ib : a.n2 - 1) * 1024 + ix) * C;
  float A[32];
#pragma unroll
  for (int r0 = 0; r0 < 32; r0 += 4) {
    float u[4][C], w[4][C];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int ch = 0; ch < C; ++ch) {
        u[k][ch] = p1[(r0 + k) * 32 * C + ch];
        w[k][ch] = p2[(r0 + k) * 32 * C + ch];
      }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float sd = 0.f;
#pragma unroll
      for (int ch = 0; ch < C; ++ch) sd = __builtin_fmaf(u[k][ch], w[k][ch], sd);
      A[r0 + k] = sd * a.seed_scale;
    }
  }
  // (the first layer, signed, stands before the loop: as a branch inside it
  // costs a copy of the tile per layer)
  cv32_layer<true, BIAS>(A, c, even, odd);
  for (int l = 1; l < a.D; ++l) cv32_layer<false, BIAS>(A, c, even, odd);
  cv_readout<32>(a, A, ix, ia, ib, valid);
}

template <int N, int C, bool BIAS>
__global__ __launch_bounds__(CvB<N>::THREADS) __attribute__((amdgpu_waves_per_eu(4)))
void cv_block_kernel(const CvArgs a) {
  using B = CvB<N>;
  constexpr int NN = B::NN, THREADS = B::THREADS, HALF = NN / 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float2* lds = reinterpret_cast<float2*>(smem);
  float4* lds4 = reinterpret_cast<float4*>(smem);
  const int tid = threadIdx.x;
  const int q = tid / N, ix = tid - q * N;
  const int qa = (q >> 2) & 3, qb = q & 3;
  int64_t bi, bj;
  pair_of(xcd_logical_block(), a.nb1, a.nb2, a.sym, a.T, &bi, &bj);
  const int64_t ia = bi * 4 + qa, ib = bj * 4 + qb;
  // a pair outside the block (ragged edge, or below the diagonal of a
  // symmetric diagonal block) runs on clamped images and writes nothing
  const bool valid = q < B::PAIRS && ia < a.n1 && ib < a.n2 && !(a.sym && bi == bj && qa > qb);
  const int64_t iac = ia < a.n1 ? ia : a.n1 - 1, ibc = ib < a.n2 ? ib : a.n2 - 1;

  // staging: THREADS / 8 threads per table slot (slots 0..3: images 4 bi + s
  // of x1, 4..7: images 4 bj + s - 4 of x2), each moving NV float4 of it
  constexpr int TPS = THREADS / 8, NV = (HALF + TPS - 1) / TPS;
  const int sl = tid / TPS, sj = tid - sl * TPS;
  const float4* src;
  {
    int64_t img = sl < 4 ? bi * 4 + sl : bj * 4 + (sl - 4);
    const int64_t lim = sl < 4 ? a.n1 : a.n2;
    if (img >= lim) img = lim - 1;
    src = reinterpret_cast<const float4*>(sl < 4 ? a.tab1 : a.tab2) + img * (int64_t)a.D * HALF + sj;
  }
  float4* dst = lds4 + sl * HALF + sj;
  // (plain floats: an array of float4 structs is not kept in registers)
  float pf[NV][4];
#define CV_FETCH(l)                                                                          \
  _Pragma("unroll") for (int m = 0; m < NV; ++m) if (HALF % TPS == 0 || sj + m * TPS < HALF) { \
    const float4 v = src[(int64_t)(l) * HALF + m * TPS];                                     \
    pf[m][0] = v.x;                                                                          \
    pf[m][1] = v.y;                                                                          \
    pf[m][2] = v.z;                                                                          \
    pf[m][3] = v.w;                                                                          \
  }
#define CV_STORE()                                                                           \
  _Pragma("unroll") for (int m = 0; m < NV; ++m) if (HALF % TPS == 0 || sj + m * TPS < HALF) \
      dst[m * TPS] = make_float4(pf[m][0], pf[m][1], pf[m][2], pf[m][3])

  // seed: the pixels of SR rows are requested together, then combined
  constexpr int SR = N < 4 ? N : 4;
  const float* p1 = a.x1 + (iac * NN + ix) * C;
  const float* p2 = a.x2 + (ibc * NN + ix) * C;
  float A[N];
#pragma unroll
  for (int r0 = 0; r0 < N; r0 += SR) {
    float u[SR][C], w[SR][C];
#pragma unroll
    for (int k = 0; k < SR; ++k)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        u[k][c] = p1[(r0 + k) * N * C + c];
        w[k][c] = p2[(r0 + k) * N * C + c];
      }
#pragma unroll
    for (int k = 0; k < SR; ++k) {
      float sd = 0.f;
#pragma unroll
      for (int c = 0; c < C; ++c) sd = __builtin_fmaf(u[k][c], w[k][c], sd);
      A[r0 + k] = sd * a.seed_scale;
    }
  }
  CV_FETCH(0);
  CV_STORE();
  __syncthreads();

  const float mL = ix >= 1 ? 1.f : 0.f;
  const float mR = ix + 1 < N ? 1.f : 0.f;
  const float2* c1 = lds + qa * NN + ix;
  const float2* c2 = lds + (4 + qb) * NN + ix;
  constexpr bool FULL = HALF % TPS == 0;
  for (int l = 0; l < a.D; ++l) {
    // (the last layer re-reads its own tables: always in bounds, never stored;
    // a conditional fetch would keep the registers live across the layer)
    const float4* nsrc = src + (int64_t)(l + 1 < a.D ? l + 1 : l) * HALF;
    if (l == 0)
      cv_layer<N, true, BIAS, B::RH, NV, TPS, FULL>(A, c1, c2, mL, mR, a.sb2, nsrc, sj, HALF, pf);
    else
      cv_layer<N, false, BIAS, B::RH, NV, TPS, FULL>(A, c1, c2, mL, mR, a.sb2, nsrc, sj, HALF, pf);
    if (l + 1 < a.D) {
      __syncthreads();
      CV_STORE();
      __syncthreads();
    }
  }
  cv_readout<N>(a, A, ix, ia, ib, valid);
}
#undef CV_FETCH
#undef CV_STORE

int launch_cv_prepare(const float* x1, int64_t n1, float2* tab1, const float* x2, int64_t n2, float2* tab2, int N, int C,
                      int D, double sw2, double sb2, hipStream_t s) {
  // both sets in one launch (the serial chain of a thread is most of its time:
  // 2 x 61 us one after the other at 1000 + 1030 images of 32 x 32); sets that
  // fill the chip many times over go one by one, within the grid's limit
  if (x2 && n1 + n2 > 0xfffff) {
    const int e = launch_cv_prepare(x1, n1, tab1, nullptr, 0, nullptr, N, C, D, sw2, sb2, s);
    return e ? e : launch_cv_prepare(x2, n2, tab2, nullptr, 0, nullptr, N, C, D, sw2, sb2, s);
  }
  const int64_t n = n1 + (x2 ? n2 : 0);
  if (n > 0x7fffffff) return -1;
  hipLaunchKernelGGL(cv_prepare_kernel, dim3((unsigned)n), dim3((unsigned)(N * N)), (size_t)N * N * sizeof(double), s,
                     x1, n1, x2, N, C, D, sw2, sb2, tab1, tab2);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template <int N, int C>
int launch_cv_pairs_nc(const CvArgs& a, bool bias, hipStream_t s) {
  const dim3 grid((unsigned)a.nblocks);
  if constexpr (N == 32) {
    const size_t lds = (size_t)4 * CV_PIECE * sizeof(float2);
    if (bias)
      hipLaunchKernelGGL((cv32_block_kernel<C, true>), grid, dim3(512), lds, s, a);
    else
      hipLaunchKernelGGL((cv32_block_kernel<C, false>), grid, dim3(512), lds, s, a);
  } else {
    using B = CvB<N>;
    if (bias)
      hipLaunchKernelGGL((cv_block_kernel<N, C, true>), grid, dim3(B::THREADS), B::LDS, s, a);
    else
      hipLaunchKernelGGL((cv_block_kernel<N, C, false>), grid, dim3(B::THREADS), B::LDS, s, a);
  }
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template <int N>
int launch_cv_pairs_n(const CvArgs& a, bool bias, hipStream_t s) {
  switch (a.C) {
    case 1: return launch_cv_pairs_nc<N, 1>(a, bias, s);
    case 2: return launch_cv_pairs_nc<N, 2>(a, bias, s);
    case 3: return launch_cv_pairs_nc<N, 3>(a, bias, s);
    case 4: return launch_cv_pairs_nc<N, 4>(a, bias, s);
    default: return -1;
  }
}

int launch_cv_pairs(int N, const float* x1, const float* x2, int64_t n1, int64_t n2, int sym, int T, int C, int D,
                    const float2* tab1, const float2* tab2, float* K, int64_t ldk, float sb2, float seed_scale,
                    hipStream_t s) {
  CvArgs a;
  a.x1 = x1;
  a.x2 = x2;
  a.n1 = n1;
  a.n2 = n2;
  a.sym = sym;
  a.T = T;
  a.C = C;
  a.D = D;
  a.tab1 = tab1;
  a.tab2 = tab2;
  a.K = K;
  a.ldk = ldk;
  a.sb2 = sb2;
  a.seed_scale = seed_scale;
  a.nb1 = (n1 + 3) / 4;
  a.nb2 = (n2 + 3) / 4;
  a.nblocks = pair_count(a.nb1, a.nb2, sym);
  if (a.nblocks <= 0) return 0;
  if (a.nblocks > 0x7fffffff) return -1;
  const bool bias = sb2 != 0.f;
  switch (N) {
    case 2: return launch_cv_pairs_n<2>(a, bias, s);
    case 4: return launch_cv_pairs_n<4>(a, bias, s);
    case 8: return launch_cv_pairs_n<8>(a, bias, s);
    case 16: return launch_cv_pairs_n<16>(a, bias, s);
    case 32: return launch_cv_pairs_n<32>(a, bias, s);
    default: return -1;
  }
}

}  // namespace nk
