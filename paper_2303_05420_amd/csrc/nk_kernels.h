// Kernel argument blocks and launchers shared between the HIP translation
// units of libnk and its host API.
#pragma once
#include <atomic>

#include "nk_common.h"

namespace nk {

// Dynamic LDS beyond 64 KiB has to be allowed per kernel, and per device.
// `seen` is one kernel's record of the largest size already allowed on each
// device (a zero-initialised static array of kMaxDevices in its launcher);
// devices beyond kMaxDevices are set on every call.  Returns 0 or -3.
constexpr int kMaxDevices = 64;
inline int allow_dyn_lds(const void* fn, size_t lds, std::atomic<size_t>* seen) {
  if (lds <= 64 * 1024) return 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -3;
  std::atomic<size_t>* rec = (dev >= 0 && dev < kMaxDevices) ? &seen[dev] : nullptr;
  if (rec && rec->load(std::memory_order_acquire) >= lds) return 0;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return -3;
  if (rec) {
    size_t cur = rec->load(std::memory_order_relaxed);
    while (cur < lds && !rec->compare_exchange_weak(cur, lds, std::memory_order_acq_rel)) {
    }
  }
  return 0;
}

// Compute units of the current device (0 if unknown), queried once per device.
inline int cu_count() {
  static std::atomic<int> counts[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
  if (dev < kMaxDevices) {
    const int c = counts[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 0;
  if (dev < kMaxDevices) counts[dev].store(n, std::memory_order_relaxed);
  return n;
}

struct PrepArgs {
  const float* x1;    // images NHWC; n1 of them, then those of x2
  const float* x2;
  int64_t n1;
  int64_t first;      // first image of this launch (of the two sets taken together)
  int64_t img_floats;
  NetDesc net;
  float2* tab1;       // table_len float2 per image
  float2* tab2;
  double* scratch;    // scratch_per_img doubles per image of the launch
  int64_t scratch_per_img;
};

// One Gram tile of a batched pass, in device memory.  Its pairs are global
// pairs [p_begin, p_begin + pair_count(n1, n2, sym)) of the pass; its images'
// tables are rows t1 + a and t2 + b of the pass's table array.
struct TileDesc {
  int64_t p_begin;
  int64_t n1, n2;
  int64_t t1, t2;
  const float* x1;
  const float* x2;
  float* K;
  int64_t ldk;
  int sym, pad;
};

struct StageArgs {
  int64_t n1, n2;
  int sym, T;
  int64_t p0, np;  // chunk = pairs [p0, p0 + np) of the block order
  const TileDesc* tiles;  // batched pass: tile table (NULL: one block given by n1, n2, x1, x2, K)
  int ntiles;
  int persist;     // > 0: grid of `persist` workgroups looping over the chunk
  int parts;       // workgroups that share a pair's sweep (32x32 pooling and 64x64 stages, set by their launchers)
  const float* x1;
  const float* x2;
  const float2* tab1;
  const float2* tab2;
  int tablen, taboff;
  int C, D;
  float sb2, seed_scale;
  int64_t img_floats;  // floats per input image (H W C): the tangent kernel compares the two images of a pair
  const float* in;  // [np][N][N][N][N]      (stages after the first)
  float* out;       // [np][N/2][N/2][N/2][N/2] (pooling stages)
  float* K;         // final stage (NULL: not written)
  int64_t ldk;
  // tangent kernel (NTK launches only): the carried C tiles in and out, the
  // NTK block (same ldk), kappa / 2 of each layer of the stage
  const float* in2;
  float* out2;
  float* K2;
  float kh[NK_MAX_DEPTH];
};

struct StageBwdArgs {
  int64_t n1, n2;
  int sym, T;
  int64_t p0, np;
  const float* x1;
  const float* x2;
  const float2* tab1;
  const float2* tab2;
  int tablen, taboff;
  int C, D;
  float sb2, seed_scale;
  int64_t img_floats;  // floats per input image (H W C), for the identical-image test of a pair
  const float* in;    // stage input [np][N]^4 (stages after the first)
  const float* gin;   // adjoint of the next stage's input [np][N/2]^4 (all but the last stage)
  float* gout;        // adjoint of this stage's input [np][N]^4 (stages after the first)
  const float* dK;    // cotangent of the block (last stage)
  int64_t lddk;
  int last;           // 1 for the last stage (adjoint from dK), else from gin
  double* W1;         // per image w sums, table layout [img][tablen]
  double* W2;
  double* xbar1;      // per image seed gradients [img][N N C] (first stage)
  double* xbar2;
  int xj;             // 1: accumulate xbar2; 0: x2's seed gradients are not wanted (xbar2 may be null at 32x32)
  int dk_t;           // 1: dK is stored transposed, dK[x2 row * lddk + x1 row]
  double* sums;       // [0]: sigma_w2 * dL/dsigma_w2 terms, [1]: dL/dsigma_b2 terms
};

struct PrepRevArgs {
  PrepArgs fwd;       // images, network and scratch (no tables)
  const double* W1;   // w sums [image][tablen]
  const double* W2;
  int tablen;
  double* xbar1;      // += image gradients [image][H W C]
  double* xbar2;
  double* sums;
};

struct FcArgs {
  const float* x1;
  const float* x2;
  int64_t n1, n2;
  int d, depth;
  float sw2, sb2;
  const float* d1;  // first-layer diagonals
  const float* d2;
  float* K;
  int64_t ldk;
  int sym;  // x1 and x2 are the same images: upper-triangle tiles, mirrored
};

// Workgroups that share the sweep of a pair's N displacement rows (N = 32, 64).
// A workgroup takes one CU (or half of one) for the N tiles of a tile column,
// so a chunk of fewer pairs than the chip holds (`resident`) leaves CUs idle; a
// part of N / 2P coarse rows costs N / P tiles, one more to begin with, and
// about two tiles' time to fill LDS.  P is the power of two with the fewest
// rounds x tiles (from four rounds on the last one no longer matters).  Whole
// calls: Myrtle-10 at 32x32x3, 2 x 60 pairs, 548 us with a workgroup a pair,
// 387 us with two; Myrtle at 64x64x3, depth 2,2,2, 1 x 20 pairs 5.85 -> 1.11 ms,
// 2 x 60 pairs 6.13 -> 3.39 ms.
inline int sweep_parts(int64_t np, int64_t resident, int N) {
  int best = 1;
  int64_t least = 0;
  for (int P = 1; P <= N / 2; P *= 2) {
    const int64_t cost = (np * P + resident - 1) / resident * (N / P + (P > 1 ? 3 : 2));
    if (P == 1 || cost < least) {
      least = cost;
      best = P;
    }
  }
  return best;
}


// Variance tables of both image sets (x2 NULL: one set).  Scratch: slots x
// prep_scratch_doubles(net) doubles, slots = prep_slots(images) images at a time.
constexpr int64_t kPrepSlots = 2048;
int64_t prep_scratch_doubles(const NetDesc& net);
int64_t prep_slots(int64_t n);
int launch_prepare_stages(const PrepArgs& a, int64_t cnt, int stages, hipStream_t stream);  // stages 0 .. stages - 1
int launch_prepare(const float* x1, int64_t n1, float2* tab1, const float* x2, int64_t n2, float2* tab2,
                   const NetDesc& net, double* scratch, int64_t slots, hipStream_t stream);
size_t stage_lds_bytes(int N, int D, bool pool, bool seed);
// ppm: pairs-per-workgroup multiplier (1 or 2) of the stage kernels of tiles
// of at most 16 x 16 (a kernel-shape choice of the batched pass; results do
// not depend on it); ignored for larger tiles.
int launch_stage(int N, const StageArgs& a, bool seed, bool pool, bool bias, hipStream_t s, int ppm = 1);
// first stage at 64x64 (seed, D <= 2 layers, pool; plain blocks only)
size_t stage64_lds_bytes(int D, int C);
int launch_stage64(const StageArgs& a, bool bias, hipStream_t s);
size_t stage_ntk_lds_bytes(int N, int D, bool pool, bool seed);
int launch_stage_ntk(int N, const StageArgs& a, bool seed, bool pool, bool bias, hipStream_t s);
int prime_stage(int N, int D, bool seed, bool pool, bool bias, int C, int ppm = 1);  // kernel attributes, no launch
int launch_put_tiles(const TileDesc* host, int n, TileDesc* dst, hipStream_t stream);
int stage_occupancy(int N, int D, bool seed, bool pool, bool bias, int C, int ppm = 1);  // resident workgroups per CU
int stage_pairs_per_wg(int N, bool pool, int ppm);  // pairs per workgroup of the stage kernel
// the 32x32 pooling stage with two tile columns per lane (stage32.hip)
size_t stage32_lds_bytes(int D, bool seed);
int launch_stage32(const StageArgs& a, bool seed, bool bias, hipStream_t s);
int stage32_occupancy(int D, bool seed, bool bias, int C);
int launch_fc(const FcArgs& a, float* d1, float* d2, hipStream_t stream);
size_t stage_bwd_lds_bytes(int N, int D, bool seed);
int launch_stage_bwd(int N, const StageBwdArgs& a, bool seed, hipStream_t s);
int launch_stage_bwd_32(const StageBwdArgs& a, bool seed, hipStream_t s);
int launch_stage_bwd_16(const StageBwdArgs& a, bool seed, hipStream_t s);
int launch_stage_bwd_small(int N, const StageBwdArgs& a, bool seed, hipStream_t s);
// Reverse of the self recursions of both image sets (x2 NULL: one set).
// Scratch: slots x prep_bwd_scratch_doubles(net) doubles, slots =
// prep_bwd_slots(images) images at a time.
constexpr int64_t kPrepBwdSlots = 512;
int64_t prep_bwd_scratch_doubles(const NetDesc& net);
int64_t prep_bwd_slots(int64_t n);
int launch_prepare_bwd(const float* x1, int64_t n1, const double* W1, double* xbar1, const float* x2, int64_t n2,
                       const double* W2, double* xbar2, const NetDesc& net, double* sums, double* scratch,
                       int64_t slots, hipStream_t stream);
int launch_cast_grad(const double* src, float* dst, int64_t n, hipStream_t s);
int launch_finish_sigma(const double* sums, double sw2, float* dsigma, hipStream_t s);
// out (cols x rows) = in^T (rows x cols), both dense; rows <= 65535 * 32.
int launch_transpose_f32(const float* in, int64_t rows, int64_t cols, float* out, hipStream_t s);
int launch_zero_f64(double* p, int64_t n, hipStream_t s);
// Diagonal entry of a matrix to be factored: an infinite one (a kernel value
// past float32) counts as 1e300, so that its unknown comes out as 0 and it takes
// no part in the others, as when dividing by its root; the factorisation works
// with reciprocals, which would make it NaN.
__device__ inline double chol_diagonal(double v) { return v > 1e300 ? 1e300 : v; }

// Cholesky factor of A (n x n, lower triangle) in place; info[0] = 1 at a
// pivot that is not positive.  Z (n x c, row-major; NULL: none) <- L^{-1} Z.
int launch_cholesky(double* A, int64_t n, int* info, double* Z, int64_t c, hipStream_t s);
// X = L^{-1} Z and X = L^{-T} Z (n x c each) for the factor that
// launch_cholesky left in A; X is another array than Z, which is used up.
int launch_chol_forward(const double* A, int64_t n, double* Z, int64_t c, double* X, hipStream_t s);
int launch_chol_backward(const double* A, int64_t n, double* Z, int64_t c, double* X, hipStream_t s);
int launch_krr_build(const float* K, int64_t n, double ridge_rel, double lam_abs, double* mean, double* A,
                     int* info, hipStream_t s);
int launch_krr_mse_bwd(const float* Kts, int64_t m, int64_t n, const double* alpha, int64_t c, const float* Yt,
                       double* G, double* sq, double* loss, double* B, hipStream_t s);
int launch_krr_outer(const double* U, int64_t rows, const double* V, int64_t cols, int64_t c, double scale,
                     float* out, hipStream_t s);

// Event bracket around one launch (the host API times the product that
// dominates a conjugate-gradient iteration through it).
struct ProfHook {
  virtual void begin(hipStream_t s) = 0;
  virtual void end(hipStream_t s) = 0;
  virtual ~ProfHook() {}
};

// One preconditioned conjugate-gradient solve (pcg.hip).  All arrays are
// device memory; n x C blocks are row-major with leading dim C.
struct PcgArgs {
  const float* K;
  int64_t n, ldk;
  const double* Y;  // n x ldy, columns c0 .. c0 + C of this group
  int64_t ldy;
  double* Xout;     // n x ldx
  int64_t ldx;
  double lam, tol;
  int max_iter;
  int r;                 // preconditioner rank (0: Ph = lam I)
  const double* Ur;      // n x r, row major: L R^{-T}, R R^T = lam I + L^T L
  double* W;             // r x 16
  double* wpart;         // lt_splits x r x 16
  int lt_splits;
  double *R, *X, *Z, *P, *Q;  // n x 16
  double* kpart;              // kmv_splits(n) x n x 16
  double *part1, *part2;      // ceil(n / 64) x 16 (per-workgroup partial sums)
  double *gamma, *ynorm, *relres;         // 2 x 16, 16, 16
  int *active, *iters;                    // 2 x 16, 16
  int* any;                               // 2 device ints: some column still iterates
  int* host_any;                          // 3 ints of pinned host memory
  ProfHook* hook;
};

// maxima: workgroups that pv and pi have room for (two entries each), at least ceil(n / 256)
int launch_pchol(const float* K, int64_t n, int64_t ldk, int rank, double pivot_tol, double* L, int* piv,
                 double* d, double* pv, int* pi, int64_t maxima, double* dpiv, hipStream_t s);
int launch_pc_setup(double* LU, int64_t n, int r, double lam, double* Ur, double* M, int* info, hipStream_t s);
int launch_pcg_group(const PcgArgs& a, int64_t c0, int C, hipStream_t s);
int kmv_splits(int64_t n);  // row splits that a product's workspace holds for 16 columns
int launch_kmv(const float* K, int64_t n, int64_t ldk, const double* P, int C, double lam, double* part, double* Q,
               double* pq_part, hipStream_t s, ProfHook* hook);
int launch_diag_mean(const float* K, int64_t n, int64_t ldk, double* out, hipStream_t s);

// Dense float64 helpers of the solvers (dense.hip).  GEMM: C (M x N, ldc) =
// beta C + alpha op(A) B, op(A) = A (M x K) or A^T (A is K x M); comp rounds
// the sums once (compensated).  -1: a form that is not compiled.
// top_a, top_b (NULL: found on the way): dn_column_top of A and B.
int dn_gemm_ff(const float* A, int64_t lda, bool a_t, const float* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
               int64_t N, int64_t K, double alpha, double beta, bool comp, hipStream_t s, const unsigned* top_a = nullptr,
               const unsigned* top_b = nullptr);
// Largest magnitude in each column of A (n x r) as the compensated products
// take it (r + 1 words of room).
int dn_column_top(const float* A, int64_t lda, int64_t n, int64_t r, unsigned* top, hipStream_t s);
int dn_gemm_fd(const float* A, int64_t lda, bool a_t, const double* B, int64_t ldb, double* C, int64_t ldc,
               int64_t M, int64_t N, int64_t K, double alpha, double beta, bool comp, hipStream_t s);
int dn_gemm_dd(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc, int64_t M,
               int64_t N, int64_t K, double alpha, double beta, hipStream_t s);
// C (float) = A B
int dn_gemm_fdf(const float* A, int64_t lda, const double* B, int64_t ldb, float* C, int64_t ldc, int64_t M,
                int64_t N, int64_t K, hipStream_t s);
// M (r x r) = lam I + L^T L, compensated, L n x r column-major; clears info[0]
int dn_ltl(const double* L, int64_t n, int64_t r, double lam, double* M, int* info, hipStream_t s);
int dn_load_shift(const float* S, int64_t lds, int64_t n, double shift, double* D, int* info, hipStream_t s);
int dn_shift(double* D, int64_t n, double shift, int* info, hipStream_t s);
int dn_identity(double* I, int64_t n, hipStream_t s);
int dn_copy_f(const float* in, int64_t ldi, int64_t rows, int64_t cols, bool trans, double* out, int64_t ldo,
              hipStream_t s);
int dn_residual_scale(const float* Y, int64_t ldy, int64_t n, int64_t c, double scale, double* X, hipStream_t s);
int dn_cast(const double* in, int64_t rows, int64_t cols, float* out, int64_t ldo, hipStream_t s);
int dn_axpby(double* D, const double* E, int64_t n, double alpha, double beta, hipStream_t s);

// CNN-VEC NNGP (cv.hip): per-image tables [img][layer][pixel] float2 of both
// sets (x2 NULL: one set), then one N-lane segment per pair.
int launch_cv_prepare(const float* x1, int64_t n1, float2* tab1, const float* x2, int64_t n2, float2* tab2, int N, int C,
                      int D, double sw2, double sb2, hipStream_t s);
int launch_cv_pairs(int N, const float* x1, const float* x2, int64_t n1, int64_t n2, int sym, int T, int C, int D,
                    const float2* tab1, const float2* tab2, float* K, int64_t ldk, float sb2, float seed_scale,
                    hipStream_t s);

}  // namespace nk
