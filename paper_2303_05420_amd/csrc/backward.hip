// Adjoint of the Myrtle NNGP (gradients with respect to the input images and
// both sigmas), hand-written reverse mode of the forward in stage.hip and
// prepare.hip.  The cross-pair stage adjoints are in stage_bwd.h (one
// translation unit per tile side); this file holds the reverse of the self
// recursions and the small kernels around them.
//
// Every scale that is proportional to sigma_w2 (conv and readout factors
// kappa, the seed scale) contributes g out / sigma_w2 to d/dsigma_w2, every
// bias term contributes v_bar to d/dsigma_b2.  J1' = 1 - acos(rho) / pi uses
// the acos fit of nk_common.h; nothing differentiates sqrt or acos at rho = 1.
//
// Self recursions (prep_rev_*, float64).  The variance maps are the output of
// the reduced self recursion of prepare.hip; it is reversed stage by stage
// with the ReLU partials
//   dF/ds = (pi - t)/(2 pi),  dF/dq = sin t sqrt(q'/q) / (4 pi)
// on the slices, the box chains of the diagonal, the pools and the seed.
// Per stage, one launch with a workgroup per kept slice (it re-runs the
// slice's layers from the stage input into LDS and reverses them; a slice
// delta != 0 stands for -delta too, whose contributions are the same, and
// counts twice) and one launch with a workgroup per image for the diagonal
// chain.  The slices of an image meet in its q_bar maps and image gradients
// through float64 atomic adds, one per pixel, layer and slice.  As in the
// forward, latency of the acos / sqrt chain is the bound: a workgroup per
// image that walked all slices through global scratch took 4.75 ms for sets
// of 20 and 100 images at Myrtle-5 32x32, these launches take 0.50 ms
// together (slices 0.29, their forward inputs 0.17, chains 0.03).
#include "prep.h"
#include "stage_bwd.h"

namespace nk {

// Per image: the stage inputs of prepare.hip, q_bar maps (table layout), and
// the adjoints of the kept slices of the stage inputs.
__host__ __device__ inline int64_t rev_qbar_off(const NetDesc& net) { return prep_off(net, net.S); }

__host__ __device__ inline int64_t rev_slices_off(const NetDesc& net, int s) {
  int64_t t = prep_off(net, net.S) + table_len(net);
  for (int k = 1; k < s; ++k) t += (int64_t)prep_half(prep_R(net, k)) * stage_res(net, k) * stage_res(net, k);
  return t;
}

int64_t prep_bwd_scratch_doubles(const NetDesc& net) { return (rev_slices_off(net, net.S) + 31) & ~31LL; }

int64_t prep_bwd_slots(int64_t n) { return n < kPrepBwdSlots ? n : kPrepBwdSlots; }

// accw and accb of the workgroup into sums, one atomic add each.
__device__ inline void rev_sums(double accw, double accb, double* __restrict__ sums) {
  __shared__ double part[2][16];
  for (int off = 32; off >= 1; off >>= 1) {
    accw += __shfl_xor(accw, off);
    accb += __shfl_xor(accb, off);
  }
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 0) {
    part[0][w] = accw;
    part[1][w] = accb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int k = 0; k < nw; ++k) {
      a += part[0][k];
      b += part[1][k];
    }
    atomicAdd(&sums[0], a);  // sum of s_bar (s - b) = sigma_w2 * d/dsigma_w2 contributions
    atomicAdd(&sums[1], b);
  }
}

// Reverse of one kept slice of a pooling stage s (maps of at most 32 x 32).
// (THREADS as in prepare_stage_kernel: two workgroups per CU for the larger maps)
template <int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS > 256 ? 8 : 4))) void
prep_rev_slice_kernel(const PrepRevArgs args, const int s, const int units) {
  extern __shared__ double rev_sm[];
  const PrepArgs& fa = args.fwd;
  const NetDesc& net = fa.net;
  const int img = blockIdx.x / units, h = blockIdx.x - img * units;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t gi = fa.first + img;
  const bool second = gi >= fa.n1;
  const float* x = second ? fa.x2 + (gi - fa.n1) * fa.img_floats : fa.x1 + gi * fa.img_floats;
  double* sc = fa.scratch + (int64_t)img * fa.scratch_per_img;
  const double* in = sc + prep_off(net, s);
  double* qbar = sc + rev_qbar_off(net) + table_off(net, s);
  const double c = (double)net.sw2 / 9.0, b = (double)net.sb2;
  const int n = stage_res(net, s), n2 = n * n, lg = 31 - __clz(n), D = net.depth[s], R = prep_R(net, s);
  int dyi, dxi;
  prep_delta(h, R, &dyi, &dxi);
  const double wgt = h == 0 ? 1.0 : 2.0;
  const int dlt = dyi * n + dxi;
  double* wA = rev_sm;
  double* wB = wA + n2;
  double* wC = wB + n2;
  double* q = wC + n2;
  double* tape = q + D * n2;
  // i + delta and i - delta inside the image
  auto fwd_ok = [&](int i) {
    const int y = (i >> lg) + dyi, xx = (i & (n - 1)) + dxi;
    return y >= 0 && y < n && xx >= 0 && xx < n;
  };
  auto back_ok = [&](int i) {
    const int y = (i >> lg) - dyi, xx = (i & (n - 1)) - dxi;
    return y >= 0 && y < n && xx >= 0 && xx < n;
  };
  for (int i = tid; i < n2; i += nt) wA[i] = prep_input(fa, x, in, s, n, i, 0, 0);
  __syncthreads();
  prep_variances(wA, q, n, lg, D, c, b);

  // forward, keeping the pre-activations
  for (int i = tid; i < n2; i += nt) wA[i] = fwd_ok(i) ? prep_input(fa, x, in, s, n, i, dyi, dxi) : 0.0;
  __syncthreads();
  for (int l = 0; l < D; ++l) {
    for (int i = tid; i < n2; i += nt) {
      double v = 0.0, sg = 0.0;
      if (fwd_ok(i)) {
        sg = c * box9(wA, n, i >> lg, i & (n - 1)) + b;
        if (l + 1 < D) v = relu_map64(sg, q[l * n2 + i], q[l * n2 + i + dlt]);
      }
      tape[l * n2 + i] = sg;
      wB[i] = v;
    }
    __syncthreads();
    double* t = wA;
    wA = wB;
    wB = t;
  }

  // adjoint of the slice's stage output, from the pooled slices
  {
    const int Rn = prep_R(net, s + 1), nn = n >> 1;
    const double* pb = sc + rev_slices_off(net, s + 1);
    for (int i = tid; i < n2; i += nt) {
      double v = 0.0;
      if (fwd_ok(i)) {
        const int y = i >> lg, xx = i & (n - 1);
        const int IY = y >> 1, IX = xx >> 1, DY = ((y + dyi) >> 1) - IY, DX = ((xx + dxi) >> 1) - IX;
        if (DY >= -Rn && DY <= Rn && DX >= -Rn && DX <= Rn) {
          bool neg;
          const int hn = prep_slice(DY, DX, Rn, &neg);
          const int I = IY * nn + IX;
          v = pb[(int64_t)hn * nn * nn + (neg ? I + DY * nn + DX : I)] / 16.0;
        }
      }
      wA[i] = v;
    }
  }
  __syncthreads();

  double accw = 0.0, accb = 0.0;
  for (int l = D - 1; l >= 0; --l) {
    const double* ql = q + l * n2;
    const double* tp = tape + l * n2;
    // sigma_bar, and the two sides' q_bar
    for (int i = tid; i < n2; i += nt) {
      double sgb = 0.0, q1 = 0.0, q2 = 0.0;
      if (fwd_ok(i)) {
        double d0, d1, d2;
        relu_partials64(tp[i], ql[i], ql[i + dlt], &d0, &d1, &d2);
        sgb = wA[i] * d0;
        q1 = wA[i] * d1;
        q2 = wA[i] * d2;
        accw += wgt * sgb * (tp[i] - b);
        accb += wgt * sgb;
      }
      wB[i] = sgb;
      wC[i] = q2;
      wA[i] = q1;
    }
    __syncthreads();
    for (int i = tid; i < n2; i += nt) {
      const double g = wA[i] + (back_ok(i) ? wC[i - dlt] : 0.0);
      atomicAdd(&qbar[l * n2 + i], wgt * g);
      wA[i] = fwd_ok(i) ? c * box9(wB, n, i >> lg, i & (n - 1)) : 0.0;
    }
    __syncthreads();
  }
  // wA = adjoint of the stage-input slice
  if (s == 0) {
    const int C = net.C;
    double* xbar = second ? args.xbar2 + (gi - fa.n1) * fa.img_floats : args.xbar1 + gi * fa.img_floats;
    for (int i = tid; i < n2; i += nt) {
      const bool f = fwd_ok(i), k = back_ok(i);
      const double g1 = f ? wA[i] : 0.0, g2 = k ? wA[i - dlt] : 0.0;
      const int i1 = f ? i + dlt : i, i2 = k ? i - dlt : i;
      for (int ch = 0; ch < C; ++ch)
        atomicAdd(&xbar[i * C + ch], wgt * (g1 * (double)x[i1 * C + ch] + g2 * (double)x[i2 * C + ch]) / C);
    }
  } else {
    double* o = sc + rev_slices_off(net, s) + (int64_t)h * n2;
    for (int i = tid; i < n2; i += nt) o[i] = wA[i];
  }
  rev_sums(accw, accb, args.sums);
}

// Reverse of the diagonal chain of stage s, q_1 = c box(base) + b, q_{l+1} =
// c box(q_l / 2) + b, after the stage's slices; one workgroup per image.
__global__ __launch_bounds__(1024) void prep_rev_chain_kernel(const PrepRevArgs args, const int s) {
  extern __shared__ double rev_sm[];
  const PrepArgs& fa = args.fwd;
  const NetDesc& net = fa.net;
  const int img = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
  const int64_t gi = fa.first + img;
  const bool second = gi >= fa.n1;
  const float* x = second ? fa.x2 + (gi - fa.n1) * fa.img_floats : fa.x1 + gi * fa.img_floats;
  const double* W = (second ? args.W2 + (gi - fa.n1) * (int64_t)args.tablen : args.W1 + gi * (int64_t)args.tablen) +
                    table_off(net, s);
  double* sc = fa.scratch + (int64_t)img * fa.scratch_per_img;
  const double* in = sc + prep_off(net, s);
  const double* qbar = sc + rev_qbar_off(net) + table_off(net, s);
  const double c = (double)net.sw2 / 9.0, b = (double)net.sb2;
  const int n = stage_res(net, s), n2 = n * n, lg = 31 - __clz(n), D = net.depth[s];
  double* w = rev_sm;
  double* g = w + n2;
  double* q = g + n2;
  for (int i = tid; i < n2; i += nt) w[i] = prep_input(fa, x, in, s, n, i, 0, 0);
  __syncthreads();
  prep_variances(w, q, n, lg, D, c, b);
  double accw = 0.0, accb = 0.0;
  // g = q_bar of layer l: the tables' and the slices' share, and that of layer l + 1
  for (int i = tid; i < n2; i += nt) w[i] = 0.0;
  __syncthreads();
  for (int l = D - 1; l >= 0; --l) {
    for (int i = tid; i < n2; i += nt) {
      const double qv = q[l * n2 + i];
      const double v = (qv > 0.0 ? W[l * n2 + i] / (2.0 * qv) : 0.0) + qbar[l * n2 + i] + w[i];
      accw += v * (qv - b);
      accb += v;
      g[i] = v;
    }
    __syncthreads();
    for (int i = tid; i < n2; i += nt) w[i] = (l > 0 ? 0.5 * c : c) * box9(g, n, i >> lg, i & (n - 1));
    __syncthreads();
  }
  // w = adjoint of the base map (0 without layers)
  if (s == 0) {
    const int C = net.C;
    double* xbar = second ? args.xbar2 + (gi - fa.n1) * fa.img_floats : args.xbar1 + gi * fa.img_floats;
    for (int i = tid; i < n2; i += nt)
      for (int ch = 0; ch < C; ++ch) xbar[i * C + ch] += 2.0 * w[i] * (double)x[i * C + ch] / C;
  } else {
    double* o = sc + rev_slices_off(net, s);
    for (int i = tid; i < n2; i += nt) o[i] = (s + 1 < net.S ? o[i] : 0.0) + w[i];
  }
  rev_sums(accw, accb, args.sums);
}

// dx (float) = xbar (double) over n images
__global__ __launch_bounds__(256) void cast_grad_kernel(const double* __restrict__ src, float* __restrict__ dst,
                                                        int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n) dst[e] = (float)src[e];
}

__global__ void finish_sigma_kernel(const double* __restrict__ sums, double sw2, float* __restrict__ dsigma) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    dsigma[0] = (float)(sums[0] / sw2);
    dsigma[1] = (float)sums[1];
  }
}

__global__ __launch_bounds__(256) void zero_f64_kernel(double* __restrict__ p, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < n) p[e] = 0.0;
}

size_t stage_bwd_lds_bytes(int N, int D, bool seed) {
  switch (N) {
    case 2: return BCfg<2>::PPWG * bwd_slot_lds_bytes<2>(D, seed);
    case 4: return BCfg<4>::PPWG * bwd_slot_lds_bytes<4>(D, seed);
    case 8: return BCfg<8>::PPWG * bwd_slot_lds_bytes<8>(D, seed);
    case 16: return BCfg<16>::PPWG * bwd_slot_lds_bytes<16>(D, seed);
    case 32: return BCfg<32>::PPWG * bwd_slot_lds_bytes<32>(D, seed);
  }
  return 0;
}

int launch_stage_bwd(int N, const StageBwdArgs& a, bool seed, hipStream_t s) {
  if (N == 32) return launch_stage_bwd_32(a, seed, s);
  if (N == 16) return launch_stage_bwd_16(a, seed, s);
  return launch_stage_bwd_small(N, a, seed, s);
}

int launch_prepare_bwd(const float* x1, int64_t n1, const double* W1, double* xbar1, const float* x2, int64_t n2,
                       const double* W2, double* xbar2, const NetDesc& net, double* sums, double* scratch,
                       int64_t slots, hipStream_t stream) {
  static std::atomic<size_t> seen_s[kMaxDevices], seen_c[kMaxDevices];
  PrepRevArgs a;
  a.fwd.x1 = x1;
  a.fwd.x2 = x2;
  a.fwd.n1 = n1;
  a.fwd.net = net;
  a.fwd.img_floats = (int64_t)net.hw * net.hw * net.C;
  a.fwd.tab1 = a.fwd.tab2 = nullptr;
  a.fwd.scratch = scratch;
  a.fwd.scratch_per_img = prep_bwd_scratch_doubles(net);
  a.W1 = W1;
  a.W2 = W2;
  a.tablen = table_len(net);
  a.xbar1 = xbar1;
  a.xbar2 = xbar2;
  a.sums = sums;
  const int64_t n = n1 + (x2 ? n2 : 0);
  for (int64_t at = 0; at < n; at += slots) {
    a.fwd.first = at;
    const int64_t cnt = n - at < slots ? n - at : slots;
    if (launch_zero_f64(scratch, cnt * a.fwd.scratch_per_img, stream)) return -3;
    if (launch_prepare_stages(a.fwd, cnt, net.S - 1, stream)) return -3;
    for (int s = net.S - 1; s >= 0; --s) {
      const int m = stage_res(net, s) * stage_res(net, s), D = net.depth[s];
      if (s + 1 < net.S) {
        const int units = prep_half(prep_R(net, s));
        const size_t lds = (size_t)(3 + 2 * D) * m * sizeof(double);
        const dim3 grid((unsigned)(cnt * units)), block((unsigned)prep_threads(m));
        if (block.x > 256) {
          if (allow_dyn_lds((const void*)prep_rev_slice_kernel<1024>, lds, seen_s)) return -3;
          hipLaunchKernelGGL(prep_rev_slice_kernel<1024>, grid, block, lds, stream, a, s, units);
        } else {
          hipLaunchKernelGGL(prep_rev_slice_kernel<256>, grid, block, lds, stream, a, s, units);
        }
      }
      const size_t lds = (size_t)(2 + D) * m * sizeof(double);
      if (allow_dyn_lds((const void*)prep_rev_chain_kernel, lds, seen_c)) return -3;
      hipLaunchKernelGGL(prep_rev_chain_kernel, dim3((unsigned)cnt), dim3((unsigned)prep_threads(m)), lds, stream, a,
                         s);
      if (hipGetLastError() != hipSuccess) return -3;
    }
  }
  return 0;
}

int launch_cast_grad(const double* src, float* dst, int64_t n, hipStream_t s) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(cast_grad_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// out (cols x rows, dense) = in^T (rows x cols, dense), through a 32 x 33
// LDS tile so that both the reads and the writes are coalesced.
__global__ __launch_bounds__(256) void transpose_f32_kernel(const float* __restrict__ in, int64_t rows, int64_t cols,
                                                            float* __restrict__ out) {
  __shared__ float t[32][33];
  const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8) {
    const int64_t r = r0 + k, c = c0 + tx;
    if (r < rows && c < cols) t[k][tx] = in[r * cols + c];
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int64_t c = c0 + k, r = r0 + tx;
    if (r < rows && c < cols) out[c * rows + r] = t[tx][k];
  }
}

int launch_transpose_f32(const float* in, int64_t rows, int64_t cols, float* out, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return 0;
  if ((rows + 31) / 32 > 65535) return -1;
  hipLaunchKernelGGL(transpose_f32_kernel, dim3((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32)), dim3(256),
                     0, s, in, rows, cols, out);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_finish_sigma(const double* sums, double sw2, float* dsigma, hipStream_t s) {
  hipLaunchKernelGGL(finish_sigma_kernel, dim3(1), dim3(64), 0, s, sums, sw2, dsigma);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_zero_f64(double* p, int64_t n, hipStream_t s) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(zero_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace nk
