// Slices of the float64 self recursion, shared by its forward (prepare.hip)
// and reverse (backward.hip): which displacement slices a stage needs, where
// their pooled sums sit in an image's scratch, and the map on one of them.
#pragma once
#include "nk_kernels.h"

namespace nk {

__host__ __device__ inline int prep_R(const NetDesc& net, int s) { return (1 << (net.S - 1 - s)) - 1; }

// Slices kept of radius R: delta = 0, and one of each pair (delta, -delta).
__host__ __device__ inline int prep_half(int R) { return ((2 * R + 1) * (2 * R + 1) + 1) / 2; }

// Workgroups that share a coarse slice (by the dy of its fine slices).  At
// four stages the 25 coarse slices of the first pool fill the chip by
// themselves and one workgroup takes all nine fine slices.
__host__ __device__ inline int prep_parts(const NetDesc& net) { return net.S <= 3 ? 3 : 1; }

// Threads of a workgroup that works on maps of m pixels.
inline int prep_threads(int m) { return m < 64 ? 64 : (m > 1024 ? 1024 : m); }

// Doubles before stage s's input slices in an image's scratch: the slices of
// stages 1 .. s - 1, [part][slice][pixel] each.
__host__ __device__ inline int64_t prep_off(const NetDesc& net, int s) {
  int64_t t = 0;
  for (int k = 1; k < s; ++k) t += (int64_t)prep_parts(net) * prep_half(prep_R(net, k)) * stage_res(net, k) * stage_res(net, k);
  return t;
}

// Position of slice (dy, dx) among the kept ones; *neg where it is -delta
// that is kept.
__device__ inline int prep_slice(int dy, int dx, int R, bool* neg) {
  *neg = dy < 0 || (dy == 0 && dx < 0);
  if (*neg) {
    dy = -dy;
    dx = -dx;
  }
  return dy == 0 ? dx : 1 + R + (dy - 1) * (2 * R + 1) + dx + R;
}

__device__ inline double relu_map64(double s, double q1, double q2) {
  double qq = q1 * q2;
  if (!(qq > 0.0)) return 0.0;
  double nrm = sqrt(qq);
  double rho = s / nrm;
  rho = rho > 1.0 ? 1.0 : (rho < -1.0 ? -1.0 : rho);
  double th = acos(rho);
  return nrm * (sqrt(fmax(1.0 - rho * rho, 0.0)) + (M_PI - th) * rho) * (0.5 / M_PI);
}

// sqrt of x in [0, 1], not denormal: two Newton steps on the hardware's 1 / sqrt
// and the residual (correctly rounded but for the last bit, as sqrt() is; that
// one also scales its argument for the ends of the range).
__device__ inline double unit_sqrt64(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  const double q = x * r;
  return x > 0.0 ? fma(fma(-q, q, x), 0.5 * r, q) : 0.0;
}

// The map above on r1 = sqrt(q1), r2 = sqrt(q2).
__device__ inline double relu_map64_roots(double s, double r1, double r2) {
  const double nrm = r1 * r2;
  if (!(nrm > 0.0)) return 0.0;
  double rho = s / nrm;
  rho = rho > 1.0 ? 1.0 : (rho < -1.0 ? -1.0 : rho);
  return nrm * (unit_sqrt64(fmax(1.0 - rho * rho, 0.0)) + (M_PI - acos(rho)) * rho) * (0.5 / M_PI);
}

// Partial derivatives of relu_map64.
__device__ inline void relu_partials64(double s, double q1, double q2, double* ds, double* dq1, double* dq2) {
  const double qq = q1 * q2;
  if (!(qq > 0.0)) {
    *ds = *dq1 = *dq2 = 0.0;
    return;
  }
  double rho = s / sqrt(qq);
  rho = rho > 1.0 ? 1.0 : (rho < -1.0 ? -1.0 : rho);
  const double th = acos(rho);
  const double sn = sqrt(fmax(1.0 - rho * rho, 0.0));
  *ds = (M_PI - th) * (0.5 / M_PI);
  *dq1 = sn * sqrt(q2 / q1) * (0.25 / M_PI);
  *dq2 = sn * sqrt(q1 / q2) * (0.25 / M_PI);
}

// 3x3 box sum with zero padding over an n x n map.  The nine reads are clamped
// into the map and requested together; under a condition each they were nine
// LDS round trips in a row (tables of 62 images of a
// three-stage 32x32 net: 142 us, 128 us so).
__device__ inline double box9(const double* m, int n, int y, int x) {
  const int yy[3] = {y > 0 ? y - 1 : 0, y, y + 1 < n ? y + 1 : y}, xx[3] = {x > 0 ? x - 1 : 0, x, x + 1 < n ? x + 1 : x};
  const bool yin[3] = {y > 0, true, y + 1 < n}, xin[3] = {x > 0, true, x + 1 < n};
  double v[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) v[k] = m[yy[k / 3] * n + xx[k % 3]];
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) s += yin[k / 3] && xin[k % 3] ? v[k] : 0.0;
  return s;
}

// The stage's variance maps q[0 .. D) (LDS), from the diagonal of its input in w0.
__device__ inline void prep_variances(const double* w0, double* q, int n, int lg, int D, double c, double b) {
  const int n2 = n * n;
  for (int l = 0; l < D; ++l) {
    const double* src = l == 0 ? w0 : q + (l - 1) * n2;
    const double f = l == 0 ? 1.0 : 0.5;
    for (int i = threadIdx.x; i < n2; i += blockDim.x) q[l * n2 + i] = c * f * box9(src, n, i >> lg, i & (n - 1)) + b;
    __syncthreads();
  }
}

// Displacement (dy, dx) of kept slice h of radius R.
__device__ inline void prep_delta(int h, int R, int* dy, int* dx) {
  if (h <= R) {
    *dy = 0;
    *dx = h;
  } else {
    *dy = 1 + (h - 1 - R) / (2 * R + 1);
    *dx = (h - 1 - R) % (2 * R + 1) - R;
  }
}

// Stage input at (pixel i, pixel i + (dy, dx)) of one image, both in the image.
__device__ inline double prep_input(const PrepArgs& a, const float* x, const double* in, int s, int n, int i, int dy,
                                    int dx) {
  const int C = a.net.C;
  const int j = i + dy * n + dx;
  if (s == 0) {
    double v = 0.0;
    for (int k0 = 0; k0 < C; k0 += 4) {
      float u[4], w[4];  // (four channels requested together)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int ch = k0 + k < C ? k0 + k : C - 1;
        u[k] = x[i * C + ch];
        w[k] = x[j * C + ch];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k0 + k < C) v += (double)u[k] * (double)w[k];
    }
    return v / C;
  }
  const int R = prep_R(a.net, s), H = prep_half(R), parts = prep_parts(a.net);
  bool neg;
  const int h = prep_slice(dy, dx, R, &neg);
  const double* p = in + (int64_t)h * n * n + (neg ? j : i);
  double v = p[0];
  if (parts == 3) {
    const double v1 = p[(int64_t)H * n * n], v2 = p[(int64_t)2 * H * n * n];
    v += v1;
    v += v2;
  }
  return v;
}

}  // namespace nk
