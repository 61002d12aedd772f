// FC NNGP block (App. A, FC listing: Flatten, depth x [Dense, ReLU], Dense).
//
//   K_1(x, x') = sigma_w2 x.x' / d + sigma_b2
//   K_{l+1}    = sigma_w2 F(K_l, K_l(x, x), K_l(x', x')) + sigma_b2
//   F(s, q, q') = sqrt(q q') / 2 J1(s / sqrt(q q'))
//
// The first layer's dot products are a dense (n1 x d) (d x n2) contraction on
// the matrix cores, and the ReLU recursion is applied in the epilogue of the
// same kernel.  The diagonals follow K_{l+1}(x, x) = sigma_w2 K_l(x, x) / 2 +
// sigma_b2 (F(q, q, q) = q/2).  Two kernels, by size (launch_fc):
//   fc_small_kernel   few outputs: a 16 x 16 tile per workgroup, its waves
//                     splitting d, fp32 matrix instructions;
//   fc_split_kernel   128 x 128 or 64 x 64 tiles, each float32 as the exact sum
//                     of three bfloat16 (bf16 matrix instructions run 16 times
//                     as fast, and six of the nine products are needed).
#include "nk_kernels.h"

namespace nk {

typedef float floatx4 __attribute__((ext_vector_type(4)));

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // rows are element aligned only
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));

// first-layer diagonals sigma_w2 |x|^2 / d + sigma_b2 of both sets, one wave per row
__global__ __launch_bounds__(256) void fc_diag_kernel(const float* __restrict__ x1, int64_t n1,
                                                      const float* __restrict__ x2, int64_t n2, int d, float sw2,
                                                      float sb2, float* __restrict__ d1, float* __restrict__ d2) {
  const int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (e >= n1 + n2) return;
  const float* p = e < n1 ? x1 + e * (int64_t)d : x2 + (e - n1) * (int64_t)d;
  double s = 0.0;
  int k = 4 * lane;
  for (; k + 3 < d; k += 256) {
    const f4u v = *reinterpret_cast<const f4u*>(p + k);
    s += (double)v.x * (double)v.x + (double)v.y * (double)v.y + (double)v.z * (double)v.z + (double)v.w * (double)v.w;
  }
  for (; k < d; ++k) s += (double)p[k] * (double)p[k];  // (the lane whose four straddle the end)
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) *(e < n1 ? d1 + e : d2 + (e - n1)) = (float)((double)sw2 * s / d + (double)sb2);
}

// The ReLU recursion and readout of one entry from its first-layer dot
// product; same: an image with itself, whose first-layer value is its diagonal
// (summed in float64; the float32 sum of squares is up to 1e-6 off at d = 384).
__device__ __forceinline__ float fc_entry(const FcArgs& a, float dot, float inv_d, float q1, float q2, bool same) {
  float k = same ? q1 : a.sw2 * dot * inv_d + a.sb2;
  for (int l = 0; l < a.depth; ++l) {
    const float qq = q1 * q2;
    const float rs = __builtin_amdgcn_rsqf(qq);
    const float rho = k * rs;
    const float f = 0.5f * (qq * rs) * (l == 0 ? j1_signed(rho) : j1_nonneg(rho));
    k = a.sw2 * (qq > 0.f ? f : 0.f) + a.sb2;
    q1 = 0.5f * a.sw2 * q1 + a.sb2;
    q2 = 0.5f * a.sw2 * q2 + a.sb2;
  }
  return k;
}

// Tile order.  Workgroups go to the 8 XCDs round-robin in launch order and
// each XCD has its own L2, so the launch index is first mapped to one
// contiguous range of tiles per XCD; each range walks the output in groups
// of FC_GROUP tile rows, column by column, so that the tiles an XCD runs at
// the same time share few x1 row tiles and x2 column tiles.  A symmetric
// block (x2 the same images as x1) runs only the tiles on and above the
// diagonal, in the pair order of the Myrtle stages over tile indices
// (groups of FC_GROUP), and each off-diagonal tile also writes its mirror.
constexpr int FC_GROUP = 8;
__device__ __forceinline__ void fc_tile(const FcArgs& a, int side, int64_t* ti, int64_t* tj) {
  const int64_t nb = gridDim.x, lin = blockIdx.x;
  const int64_t xcd = lin & 7, q = nb >> 3, rem = nb & 7;
  const int64_t id = (xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q) + (lin >> 3);
  const int64_t gy = (a.n1 + side - 1) / side, gx = (a.n2 + side - 1) / side;
  if (a.sym) {
    pair_of(id, gy, gy, 1, FC_GROUP, ti, tj);
    return;
  }
  const int64_t grp = id / (FC_GROUP * gx), first = grp * FC_GROUP;
  const int64_t rows = gy - first < FC_GROUP ? gy - first : FC_GROUP;
  const int64_t in = id - first * gx;
  *ti = first + in % rows;
  *tj = in / rows;
}

// Four entries of a column, rows rb .. rb + 3; mirror: also as row c, columns
// rb .. rb + 3; upper: only entries on and above the diagonal (a tile on the
// diagonal of a symmetric block).
__device__ __forceinline__ void fc_store4(const FcArgs& a, const float (&kv)[4], int64_t rb, int64_t c, bool mirror,
                                          bool upper) {
  if (c >= a.n2) return;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (rb + v < a.n1 && !(upper && rb + v > c)) a.K[(rb + v) * a.ldk + c] = kv[v];
  if (!mirror) return;
  float* m = a.K + c * a.ldk + rb;
  if (!upper && rb + 3 < a.n1 && (reinterpret_cast<uintptr_t>(m) & 15) == 0) {
    *reinterpret_cast<float4*>(m) = make_float4(kv[0], kv[1], kv[2], kv[3]);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (rb + v < a.n1 && !(upper && rb + v >= c)) m[v] = kv[v];
  }
}

// Few outputs.  A workgroup owns a 16 x 16 tile and its 16 waves take every
// 16th chunk of 16 features each (lane l = 16 g + i reads features 4 g .. 4 g
// + 3 of row i of both operands, one 16-byte load each), so the depth of the
// contraction is spread over a CU however few tiles there are; the squares for
// the diagonals are summed in float64 on the way, so the call is one launch.
// Bound by the reading of the longer set.  4 x 1000 at d = 3072: 10.9 us
// (two launches for the diagonals and 8 workgroups of 128 x 128 walking all of
// d: 307 us).
constexpr int FS_W = 16;
__global__ __launch_bounds__(64 * FS_W) void fc_small_kernel(const FcArgs a) {
  __shared__ float part[FS_W][256];
  __shared__ double sq[2][FS_W][16];
  __shared__ float q[2][16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  int64_t ti, tj;
  fc_tile(a, 16, &ti, &tj);
  const int64_t r0 = ti * 16, c0 = tj * 16;
  const int64_t r = r0 + i < a.n1 ? r0 + i : a.n1 - 1, c = c0 + i < a.n2 ? c0 + i : a.n2 - 1;
  const float* p1 = a.x1 + r * (int64_t)a.d;
  const float* p2 = a.x2 + c * (int64_t)a.d;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  double s1 = 0.0, s2 = 0.0;
  auto step = [&](const float (&u)[4], const float (&v)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(u[t], v[t], acc, 0, 0, 0);
      s1 = __builtin_fma((double)u[t], (double)u[t], s1);
      s2 = __builtin_fma((double)v[t], (double)v[t], s2);
    }
  };
  int k0 = 16 * w;
#pragma unroll 4
  for (; k0 + 16 <= a.d; k0 += 16 * FS_W) {
    const f4u x = *reinterpret_cast<const f4u*>(p1 + k0 + 4 * g), y = *reinterpret_cast<const f4u*>(p2 + k0 + 4 * g);
    const float u[4] = {x.x, x.y, x.z, x.w}, v[4] = {y.x, y.y, y.z, y.w};
    step(u, v);
  }
  if (k0 < a.d) {
    const int k = k0 + 4 * g;
    float u[4], v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      u[t] = k + t < a.d ? p1[k + t] : 0.f;
      v[t] = k + t < a.d ? p2[k + t] : 0.f;
    }
    step(u, v);
  }
  s1 += __shfl_xor(s1, 16);
  s2 += __shfl_xor(s2, 16);
  s1 += __shfl_xor(s1, 32);
  s2 += __shfl_xor(s2, 32);
  if (g == 0) {
    sq[0][w][i] = s1;
    sq[1][w][i] = s2;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) part[w][(4 * g + v) * 16 + i] = acc[v];
  __syncthreads();
  double dot = 0.0;
  if (tid < 256) {
    for (int m = 0; m < FS_W; ++m) dot += (double)part[m][tid];
  } else if (tid < 288) {
    const int o = (tid >> 4) & 1, e = tid & 15;
    double t = 0.0;
    for (int m = 0; m < FS_W; ++m) t += sq[o][m][e];
    q[o][e] = (float)((double)a.sw2 * t / a.d + (double)a.sb2);
  }
  __syncthreads();
  if (tid >= 256) return;
  const int64_t er = r0 + (tid >> 4), ec = c0 + (tid & 15);
  if (er >= a.n1 || ec >= a.n2 || (a.sym && ec < er)) return;
  const float kv = fc_entry(a, (float)dot, 1.0f / (float)a.d, q[0][tid >> 4], q[1][tid & 15],
                            a.sym && er == ec);
  a.K[er * a.ldk + ec] = kv;
  if (a.sym && ec > er) a.K[ec * a.ldk + er] = kv;
}

// A float32 pair as three bfloat16 pairs, x = h + m + l exactly (8 significant
// bits each; what underflows bfloat16's 2^-133 is lost).
__device__ __forceinline__ void fc_split2(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  auto pk = [](float a, float b) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f2{a, b}, bf2)); };
  auto lo = [](unsigned u) { return __builtin_bit_cast(float, u << 16); };
  auto hi = [](unsigned u) { return __builtin_bit_cast(float, u & 0xffff0000u); };
  h = pk(x0, x1);
  const float r0 = x0 - lo(h), r1 = x1 - hi(h);
  m = pk(r0, r1);
  l = pk(r0 - lo(m), r1 - hi(m));
}

// Tiles of 64 WB x 64 WB outputs, a quadrant of WB x WB blocks of 32 x 32 per
// wave on v_mfma_f32_32x32x16_bf16.  The rows of both operands are read as
// float32, split into three bfloat16 parts on the way into LDS, and the
// products h h', h m', m h', m m', h l', l h' accumulate in float32 (NP = 6);
// the three left out are below 2^-24 of the product of the two numbers (NP = 9,
// all of them, below 64 features).  They have either sign where the features of
// a row take many values; where they take few they add up, to 6e-8 of the entry
// at most, but there the roundings of the sum weigh more, and it rounds less
// often than with fp32 instructions.  Largest error against float64 of 3.3e6
// entries (normalised, no ReLU layers) at d = 64 and 3072, fp32 instructions first:
// normal features 2.2e-7, 2.4e-7 and 2.0e-7, 1.8e-7; rows of one value 1.0e-6,
// 4.6e-5 and 7.3e-7, 2.8e-5; of two values 8.9e-7, 3.8e-5 and 4.4e-7, 1.4e-5.
// Exchanged operands.  A product and its counterpart (h l' and l h', h m' and m
// h') stand in one instruction, in neighbouring registers of a lane: the 8 terms
// of a lane are summed together whatever their order (measured: no bit differs
// in 4e6 results when registers change places in both operands; a third of them
// when the two halves of the wave do), so K(x2, x1) is the transpose of K(x1,
// x2) bit for bit, and an entry's bits do not depend on where the block is cut.
// The two after one another left 2 % of the entries different.  It costs the
// moves that pair l with h and exchange one side's halves, 5 %: 7.3-7.5 ms for
// the Gram below against 6.9-7.15 (a sum per side needs no moves, but three
// accumulators do not fit the registers of two waves; the operands read from LDS
// as they are used in place of the moves: 11 %).
// Non-finite inputs: an infinity or NaN makes its row's diagonal non-finite,
// and from one ReLU on the entry no longer depends on the dot product; without
// ReLU layers such an entry's product is formed anew in float32.
// LDS: [buffer][operand], rows of 16 KT features: h and m in turn, two features
// each (plane Q), and l (plane L), rows padded by 16 bytes so that 8 lanes'
// 16-byte reads fall on different banks.  Two buffers, one
// barrier per tile of features: the next tile is split and stored while the
// current one multiplies, the one after it is on its way from memory (its
// loads stay in flight across the barrier, which waits for LDS only); two
// workgroups per CU.
// Bound: the matrix instructions, 6 x 2 n1 n2 d operations at the bf16 rate, by
// the reads that feed them.  FC-3 Gram of 20000 x 3072 (symmetric): 7.3-7.5 ms,
// about 1000 TFLOP/s of bf16 products (a large library product reaches 1081 to
// 1309 from card to card); with fp32 instructions 12.3 ms, 0.65 of their peak.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int WB, int KT, int NP>
__global__ __launch_bounds__(256, WB == 1 ? 4 : 2) void fc_split_kernel(const FcArgs a) {
  constexpr int TM = 64 * WB, BK = 16 * KT, QROW = 4 * BK + 16, LROW = 2 * BK + 16;
  constexpr int OPND = TM * (QROW + LROW), BUF = 2 * OPND;
  constexpr int TPR = BK / 4, RPP = 256 / TPR, NQ = TM / RPP;  // threads a row, rows a pass, passes an operand
  __shared__ __attribute__((aligned(16))) char lds[2 * BUF];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int64_t ti, tj;
  fc_tile(a, TM, &ti, &tj);
  const int64_t r0 = ti * TM, c0 = tj * TM;
  const bool mirror = a.sym, upper = a.sym && ti == tj;
  // staging: this thread's float4 m of either operand is row tid / TPR + RPP m,
  // features sk .. sk + 3 of the tile
  const int srow = tid / TPR, sk = 4 * (tid % TPR);
  const float* p1[NQ];
  const float* p2[NQ];
#pragma unroll
  for (int m = 0; m < NQ; ++m) {
    const int64_t r = r0 + srow + RPP * m, c = c0 + srow + RPP * m;
    p1[m] = a.x1 + (r < a.n1 ? r : a.n1 - 1) * (int64_t)a.d + sk;
    p2[m] = a.x2 + (c < a.n2 ? c : a.n2 - 1) * (int64_t)a.d + sk;
  }
  struct Regs {
    f4u a[NQ], b[NQ];
  };
  // (past the last tile: the last one again, in bounds and never stored)
  const int nt = (a.d + BK - 1) / BK;
  auto fetch = [&](int t, Regs& v) {
    const int k0 = (t < nt ? t : nt - 1) * BK;
    if (k0 + BK <= a.d) {
#pragma unroll
      for (int m = 0; m < NQ; ++m) {
        v.a[m] = *reinterpret_cast<const f4u*>(p1[m] + k0);
        v.b[m] = *reinterpret_cast<const f4u*>(p2[m] + k0);
      }
    } else {
#pragma unroll
      for (int m = 0; m < NQ; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool in = k0 + sk + q < a.d;
          v.a[m][q] = in ? p1[m][k0 + q] : 0.f;
          v.b[m][q] = in ? p2[m][k0 + q] : 0.f;
        }
    }
  };
  auto put = [&](const f4u& x, char* q, char* l) {
    unsigned h0, m0, l0, h1, m1, l1;
    fc_split2(x.x, x.y, h0, m0, l0);
    fc_split2(x.z, x.w, h1, m1, l1);
    *reinterpret_cast<uint4*>(q) = make_uint4(h0, m0, h1, m1);
    *reinterpret_cast<uint2*>(l) = make_uint2(l0, l1);
  };
  char* sq = lds + srow * QROW + 4 * sk;
  char* sl = lds + TM * QROW + srow * LROW + 2 * sk;
  auto store = [&](const Regs& v, int buf) {
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int o = buf * BUF;
      put(v.a[m], sq + o + RPP * m * QROW, sl + o + RPP * m * LROW);
      put(v.b[m], sq + o + OPND + RPP * m * QROW, sl + o + OPND + RPP * m * LROW);
    }
  };
  f16v acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  const int wr = 32 * WB * (w >> 1), wc = 32 * WB * (w & 1), li = lane & 31, kh = lane >> 5;
  const char* qa = lds + (wr + li) * QROW + 32 * kh;
  const char* la = lds + TM * QROW + (wr + li) * LROW + 16 * kh;
  const char* qb = lds + OPND + (wc + li) * QROW + 32 * kh;
  const char* lb = lds + OPND + TM * QROW + (wc + li) * LROW + 16 * kh;
  // this lane's 8 features of a row: {h, m, h, m} of features 0 .. 3 and of 4 .. 7, and l
  struct Frag {
    uint4 q[2], l;
  };
  // Features 0 .. 3 (half 0) or 4 .. 7 as one operand of an instruction: two
  // features' part x and the same two's part y, in turn; against (x, y) of one
  // side stands (y, x) of the other.
  enum { HM, HL, ML };
  auto pairs = [](const Frag& f, int half, int kind, bool other) {
    const uint4 q = f.q[half];
    const unsigned l0 = half ? f.l.z : f.l.x, l1 = half ? f.l.w : f.l.y;
    const unsigned x0 = kind == ML ? q.y : q.x, x1 = kind == ML ? q.w : q.z;
    const unsigned y0 = kind == HM ? q.y : l0, y1 = kind == HM ? q.w : l1;
    return __builtin_bit_cast(bf8, other ? make_uint4(y0, x0, y1, x1) : make_uint4(x0, y0, x1, y1));
  };
  auto product = [&](const bf8 (&x)[WB], const bf8 (&y)[WB]) {
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
      for (int j = 0; j < WB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], y[j], acc[i][j], 0, 0, 0);
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
      Frag a[WB], b[WB];
#pragma unroll
      for (int i = 0; i < WB; ++i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a[i].q[h] = *reinterpret_cast<const uint4*>(qa + buf * BUF + i * 32 * QROW + 64 * kk + 16 * h);
          b[i].q[h] = *reinterpret_cast<const uint4*>(qb + buf * BUF + i * 32 * QROW + 64 * kk + 16 * h);
        }
        a[i].l = *reinterpret_cast<const uint4*>(la + buf * BUF + i * 32 * LROW + 32 * kk);
        b[i].l = *reinterpret_cast<const uint4*>(lb + buf * BUF + i * 32 * LROW + 32 * kk);
      }
      bf8 ahm[2][WB], bhm[2][WB], bmh[2][WB], ahl[2][WB], blh[2][WB];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < WB; ++i) {
          ahm[h][i] = pairs(a[i], h, HM, false);
          bhm[h][i] = pairs(b[i], h, HM, false);
          bmh[h][i] = pairs(b[i], h, HM, true);
          ahl[h][i] = pairs(a[i], h, HL, false);
          blh[h][i] = pairs(b[i], h, HL, true);
        }
      // smallest products first
      if constexpr (NP == 9) {
        bf8 x[WB], y[WB];
#pragma unroll
        for (int i = 0; i < WB; ++i) {
          x[i] = __builtin_bit_cast(bf8, a[i].l);
          y[i] = __builtin_bit_cast(bf8, b[i].l);
        }
        product(x, y);  // l l'
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // m l', l m'
#pragma unroll
          for (int i = 0; i < WB; ++i) {
            x[i] = pairs(a[i], h, ML, false);
            y[i] = pairs(b[i], h, ML, true);
          }
          product(x, y);
        }
      }
      // (the operands formed before the first product: with the moves between
      // the products the large Gram takes 2 % longer)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < 2; ++h) product(ahl[h], blh[h]);  // h l', l h'
#pragma unroll
      for (int h = 0; h < 2; ++h) product(ahm[h], bmh[h]);  // h m', m h'
#pragma unroll
      for (int h = 0; h < 2; ++h) product(ahm[h], bhm[h]);  // h h', m m'
    }
  };
  Regs even, odd;  // the tiles of even and odd number on their way
  fetch(0, even);
  fetch(1, odd);
  store(even, 0);
  lds_barrier();
  for (int t = 0; t < nt; t += 2) {
    fetch(t + 2, even);
    multiply(0);
    store(odd, 1);  // tile t + 1
    lds_barrier();
    if (t + 1 < nt) {
      fetch(t + 3, odd);
      multiply(1);
      store(even, 0);  // tile t + 2
      lds_barrier();
    }
  }
  // lane l holds column l & 31, rows 8 (v >> 2) + 4 (l >> 5) + (v & 3) of a block
  const float inv_d = 1.0f / (float)a.d;
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j) {
      const int64_t c = c0 + wc + 32 * j + li;
      const float q2 = a.d2[c < a.n2 ? c : a.n2 - 1];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t rb = r0 + wr + 32 * i + 8 * u + 4 * kh;
        float kv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
          kv[v] = fc_entry(a, acc[i][j][4 * u + v], inv_d, a.d1[rb + v < a.n1 ? rb + v : a.n1 - 1], q2,
                           upper && rb + v == c);
        fc_store4(a, kv, rb, c, mirror, upper);
      }
    }
  if (a.depth == 0) {
    // no ReLU layer: entries of rows that hold an infinity or NaN (their
    // diagonal says so), from a plain float32 product
    __syncthreads();
    for (int e = tid; e < TM * TM; e += 256) {
      const int64_t r = r0 + e / TM, c = c0 + e % TM;
      if (r >= a.n1 || c >= a.n2 || (upper && r > c)) continue;
      if (__builtin_isfinite(a.d1[r]) && __builtin_isfinite(a.d2[c])) continue;
      float dot = 0.f;
      for (int k = 0; k < a.d; ++k) dot = __builtin_fmaf(a.x1[r * a.d + k], a.x2[c * a.d + k], dot);
      const float kv = fc_entry(a, dot, inv_d, a.d1[r], a.d2[c], upper && r == c);
      a.K[r * a.ldk + c] = kv;
      if (mirror) a.K[c * a.ldk + r] = kv;
    }
  }
}

// Tiles of side `side` that a launch has to form.
static int64_t fc_tiles(const FcArgs& a, int64_t side) {
  const int64_t t1 = (a.n1 + side - 1) / side, t2 = (a.n2 + side - 1) / side;
  return a.sym ? t1 * (t1 + 1) / 2 : t1 * t2;
}

int launch_fc(const FcArgs& a, float* d1, float* d2, hipStream_t stream) {
  // Kernel by size.  16 x 16 tiles read 16 + 16 rows for 256 outputs, four times
  // what 64 x 64 ones do, but spread any d over a CU.  Their time goes with their
  // number; that of 64 x 64 tiles is one tile's walk over d (13.8 / 31 / 87 us at
  // d = 64 / 784 / 3072, 1600 or more of the small tiles) until the chip is
  // full, and then grows by some four small tiles' time per tile.  So a block of
  // up to 16 rows, four small tiles to a large one, stays with the small ones
  // however long it is: 4 x 20000 10.7 / 17 / 45 us against 17 / 51 / 147, 4 x
  // 100000 31 / 73 / 242 against 45 / 161 / 541.  Below the line: 32 x 20000 (2500
  // small tiles) 16 / 30 / 112 against 18 / 51 / 147, 500 x 1000 (2016) 13 / 23 /
  // 94 against 14 / 32 / 92; above it: 32 x 50000 (6250) 33 / 66 / 312 against 28 /
  // 85 / 304, 300 x 2000 (2375) 15 / 29 / 118 against 14 / 33 / 96, 500 x 2000
  // (4000) 22 / 43 / 184 against 14 / 33 / 97.  A symmetric block also writes its
  // mirror, 64 bytes a row from small tiles, which shows where d is small: 900 at
  // d = 64 (1653) 18 against 14; 1000 (2016) at 784 / 3072 27 / 88 against 32 / 90.
  const int64_t small = fc_tiles(a, 16), t64 = fc_tiles(a, 64);
  if (small <= (a.sym && a.d < 384 ? 1536 : 1600 + 4 * t64)) {
    hipLaunchKernelGGL(fc_small_kernel, dim3((unsigned)small), dim3(64 * FS_W), 0, stream, a);
    return hipGetLastError() == hipSuccess ? 0 : -3;
  }
  FcArgs b = a;
  b.d1 = d1;
  b.d2 = a.sym ? d1 : d2;
  const int64_t rows = a.n1 + (a.sym ? 0 : a.n2);
  hipLaunchKernelGGL(fc_diag_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, a.x1, a.n1, a.x2,
                     a.sym ? 0 : a.n2, a.d, a.sw2, a.sb2, d1, d2);
  // 128 x 128 tiles halve the reads of 64 x 64 ones, which fill the chip sooner
  // and hide the epilogue (four workgroups a CU): 4096 x 4096 at d = 3072 / 784
  // / 64: 620 / 192 / 69 us against 760 / 218 / 58; 3000 x 3000 (576 tiles):
  // 423 / 150 / 59 against 427 / 130 / 37.
  // (A launch of 2^24 workgroups of 256 is past the grid's limit of 2^32 threads;
  // 64 x 64 tiles reach it at 275 GB of outputs.)
  const int64_t t128 = fc_tiles(a, 128);
  const bool wide = (t128 >= 640 && a.d >= 384) || t64 >= 1 << 24;
  if (wide && a.d >= 64)
    hipLaunchKernelGGL((fc_split_kernel<2, 1, 6>), dim3((unsigned)t128), dim3(256), 0, stream, b);
  else if (wide)
    hipLaunchKernelGGL((fc_split_kernel<2, 1, 9>), dim3((unsigned)t128), dim3(256), 0, stream, b);
  else if (a.d >= 64)
    hipLaunchKernelGGL((fc_split_kernel<1, 1, 6>), dim3((unsigned)t64), dim3(256), 0, stream, b);
  else
    hipLaunchKernelGGL((fc_split_kernel<1, 1, 9>), dim3((unsigned)t64), dim3(256), 0, stream, b);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace nk
