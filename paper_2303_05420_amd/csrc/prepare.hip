// Per-image variance tables for the Myrtle NNGP (float64 inside).
//
// Every ReLU of a pair (x, x') needs the variances q(i) = S_xx(i, i) and
// q'(j) of the two images at that layer: the diagonal of each image's own
// recursion (App. A Myrtle network; the ReLU map takes the two marginal
// variances and the covariance).  Inside a stage a 3x3 conv keeps the pixel
// displacement delta = j - i, and on the delta = 0 slice the ReLU map is
// F(q, q, q) = q / 2, so within a stage
//   q_1 = c box(base) + b,   q_{l+1} = c box(q_l / 2) + b,   c = sigma_w2 / 9,
// with base the diagonal of the stage input.  A 2x2 pool mixes the slices
// delta = 2 Delta + {-1, 0, 1}^2, so the diagonal after a pool needs the
// previous stage's slices |delta| <= 1, which need the stage before's
// |delta| <= 3, and so on: stage s of S uses slices |delta| <= 2^(S-1-s) - 1.
// These kernels run those slices of the self recursion (a few percent of one
// pair's work per image) and write, per stage, layer and pixel,
//   alpha = 1 / sqrt(q)         (0 where q == 0),
//   beta  = sqrt(q * kappa / 2),
// where kappa is the factor the next linear step applies to the ReLU output
// (c inside a stage, c / 16 before a pool, sigma_w2 / n^4 before the final
// global-average readout).  The pair kernels then form
// rho = S alpha(i) alpha'(j) and kappa F = beta(i) beta'(j) J1(rho).
//
// Split.  One launch per stage; a workgroup owns one coarse slice Delta of
// the next stage's input (or, for up to three stages, one dy of it) and runs
// the fine slices 2 Delta + {-1, 0, 1}^2 that feed it, its maps in LDS, the
// pooled sum in registers: no slice of the full resolution leaves the
// workgroup.  The slices of -delta are those of delta read at the other
// pixel, so only half of the coarse slices are formed.  What bounds it is the
// latency of the float64 acos / sqrt chain of one layer times the layers run
// in a row: with one workgroup per image walking all slices through global
// scratch (the first form) that chain was 49 x 3 layers long at Myrtle-10
// 32x32: a call on 2 and 60 images spent 2.28 ms here (two sets, one after
// the other), one on 8192 images 18.7 ms.  Now it is 3 x 3 layers long in 15
// workgroups per image and both sets share a launch: 0.11 ms and 8.9 ms.
#include "prep.h"

namespace nk {

int64_t prep_scratch_doubles(const NetDesc& net) { return (prep_off(net, net.S) + 31) & ~31LL; }

int64_t prep_slots(int64_t n) { return n < kPrepSlots ? n : kPrepSlots; }

// Stage s of every image of the launch: `units` workgroups per image, each
// one (coarse slice, part); the first of them also writes the stage's tables.
// THREADS = 1024 (maps of more than 256 pixels): registers for two workgroups
// per CU, which pass under each other's barriers and float64 chains (one per CU
// at 68 registers: 125 us for the tables of 62 images of Myrtle-10 at 32x32,
// two at 61: 111 us).  Smaller maps run in smaller workgroups and do not need it.
template <int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS > 256 ? 8 : 4))) void
prepare_stage_kernel(const PrepArgs args, const int s, const int units) {
  extern __shared__ double prep_sm[];
  const NetDesc& net = args.net;
  const int img = blockIdx.x / units, unit = blockIdx.x - img * units;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t gi = args.first + img;  // image of the two sets taken together
  const bool second = gi >= args.n1;
  const float* x = (second ? args.x2 + (gi - args.n1) * args.img_floats : args.x1 + gi * args.img_floats);
  double* sc = args.scratch + (int64_t)img * args.scratch_per_img;
  const double* in = sc + prep_off(net, s);
  const double c = (double)net.sw2 / 9.0, b = (double)net.sb2;
  const int n = stage_res(net, s), n2 = n * n, lg = 31 - __clz(n), D = net.depth[s];
  double* w0 = prep_sm;
  double* w1 = w0 + n2;
  double* q = w1 + n2;

  // variance maps of the stage, from the diagonal of its input
  for (int i = tid; i < n2; i += nt) w0[i] = prep_input(args, x, in, s, n, i, 0, 0);
  __syncthreads();
  prep_variances(w0, q, n, lg, D, c, b);
  if (unit == 0 && args.tab1) {
    float2* tab = (second ? args.tab2 + (gi - args.n1) * (int64_t)table_len(net)
                          : args.tab1 + gi * (int64_t)table_len(net)) + table_off(net, s);
    for (int l = 0; l < D; ++l) {
      // scale of the next linear step on this ReLU output: the next conv (c),
      // through the pools in between (1/16 each; stages without layers only
      // pool), or the global-average readout (sigma_w2 / n^4)
      double kappa = c;
      if (l + 1 == D) {
        int s2 = s + 1;
        double f = 1.0 / 16.0;
        while (s2 < net.S && net.depth[s2] == 0) {
          f /= 16.0;
          ++s2;
        }
        kappa = s2 < net.S ? c * f : (double)net.sw2 / ((double)n * n * n * n);
      }
      for (int i = tid; i < n2; i += nt) {
        const double qi = q[l * n2 + i];
        const float al = qi > 0.0 ? (float)(1.0 / sqrt(qi)) : 0.0f;
        const float be = qi > 0.0 ? (float)sqrt(qi * kappa * 0.5) : 0.0f;
        tab[l * n2 + i] = make_float2(al, be);
      }
    }
  }
  if (s + 1 == net.S) return;

  // the map below takes the roots (its own pixels, before the first barrier)
  for (int i = tid; i < n2; i += nt)
    for (int l = 0; l < D; ++l) q[l * n2 + i] = sqrt(q[l * n2 + i]);
  // the fine slices of this unit's coarse slice (DY, DX), pooled: coarse
  // pixel I of it gathers the fine pixels i = 2I + a with (i + delta) >> 1 ==
  // I + Delta in each dimension
  const int Rn = prep_R(net, s + 1), nn = n >> 1, H = prep_half(Rn), parts = prep_parts(net);
  const int h = unit / parts, part = unit - h * parts;
  int DY, DX;
  prep_delta(h, Rn, &DY, &DX);
  const int ey0 = parts == 3 ? part - 1 : -1, ey1 = parts == 3 ? part - 1 : 1;
  const int IY = tid >> (lg - 1), IX = tid & (nn - 1);  // this thread's coarse pixel (tid < nn * nn)
  const bool coarse = tid < nn * nn && IY + DY < nn && IX + DX >= 0 && IX + DX < nn;
  double acc = 0.0;
  for (int ey = ey0; ey <= ey1; ++ey)
    for (int ex = -1; ex <= 1; ++ex) {
      const int dyi = 2 * DY + ey, dxi = 2 * DX + ex;
      for (int i = tid; i < n2; i += nt) {
        const int y2 = (i >> lg) + dyi, x2 = (i & (n - 1)) + dxi;
        w0[i] = (y2 >= 0 && y2 < n && x2 >= 0 && x2 < n) ? prep_input(args, x, in, s, n, i, dyi, dxi) : 0.0;
      }
      __syncthreads();
      for (int l = 0; l < D; ++l) {
        for (int i = tid; i < n2; i += nt) {
          const int y = i >> lg, xx = i & (n - 1), y2 = y + dyi, x2 = xx + dxi;
          double v = 0.0;
          if (y2 >= 0 && y2 < n && x2 >= 0 && x2 < n)
            v = relu_map64_roots(c * box9(w0, n, y, xx) + b, q[l * n2 + i], q[l * n2 + y2 * n + x2]);
          w1[i] = v;
        }
        __syncthreads();
        double* t = w0;
        w0 = w1;
        w1 = t;
      }
      if (coarse) {
        // e = -1: the second fine pixel, e = 1: the first, e = 0: both
        double v = 0.0;
        for (int ay = ey < 0 ? 1 : 0; ay <= (ey > 0 ? 0 : 1); ++ay)
          for (int ax = ex < 0 ? 1 : 0; ax <= (ex > 0 ? 0 : 1); ++ax) v += w0[(2 * IY + ay) * n + 2 * IX + ax];
        acc += v / 16.0;
      }
      __syncthreads();
    }
  if (tid < nn * nn) sc[prep_off(net, s + 1) + ((int64_t)part * H + h) * nn * nn + tid] = acc;
}

int launch_prepare_stages(const PrepArgs& a, int64_t cnt, int stages, hipStream_t stream) {
  static std::atomic<size_t> seen[kMaxDevices];
  const NetDesc& net = a.net;
  for (int s = 0; s < stages; ++s) {
    const int m = stage_res(net, s) * stage_res(net, s);
    const int units = s + 1 < net.S ? prep_half(prep_R(net, s + 1)) * prep_parts(net) : 1;
    const size_t lds = (size_t)(2 + net.depth[s]) * m * sizeof(double);
    const dim3 grid((unsigned)(cnt * units)), block((unsigned)prep_threads(m));
    if (block.x > 256) {
      if (allow_dyn_lds((const void*)prepare_stage_kernel<1024>, lds, seen)) return -3;
      hipLaunchKernelGGL(prepare_stage_kernel<1024>, grid, block, lds, stream, a, s, units);
    } else {
      hipLaunchKernelGGL(prepare_stage_kernel<256>, grid, block, lds, stream, a, s, units);
    }
    if (hipGetLastError() != hipSuccess) return -3;
  }
  return 0;
}

int launch_prepare(const float* x1, int64_t n1, float2* tab1, const float* x2, int64_t n2, float2* tab2,
                   const NetDesc& net, double* scratch, int64_t slots, hipStream_t stream) {
  PrepArgs a;
  a.x1 = x1;
  a.x2 = x2;
  a.n1 = n1;
  a.net = net;
  a.img_floats = (int64_t)net.hw * net.hw * net.C;
  a.tab1 = tab1;
  a.tab2 = tab2;
  a.scratch = scratch;
  a.scratch_per_img = prep_scratch_doubles(net);
  const int64_t n = n1 + (x2 ? n2 : 0);
  for (int64_t at = 0; at < n; at += slots) {
    a.first = at;
    if (launch_prepare_stages(a, n - at < slots ? n - at : slots, net.S, stream)) return -3;
  }
  return 0;
}

}  // namespace nk
