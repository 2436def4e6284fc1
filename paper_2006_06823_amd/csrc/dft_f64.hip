// Truncated DFT contractions in double (v_mfma_f64_16x16x4f64).
//
// The FP64 problems are 2D ones of some ten thousand nodes, where a transform is a few hundred thousand
// operations and a launch costs more than its arithmetic: what bounds them is the number of kernels and the chain
// of latencies inside each.  So one kernel transforms both inner axes (combination, scaling and accumulation
// included), no operand is staged, a wave requests its operands at once, and the intermediate stays in registers:
// in the output layout of the matrix instruction (register r of a lane holds row 4 r + lane / 16, column
// lane % 16) a 16-column tile is already the second operand of the next product, step r taking register r.
// 64 x 64 nodes, 16 x 16 coefficients, one field: inclusion 19 -> 3.7 us, projection 35 -> 4.2 us, against
// LDS-staged vector-unit products with one launch per axis and one per combination.
#include "kernels.h"
#include "prof.h"

#include <algorithm>
#include <string>

namespace lddmm {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// p[i] where ok, else zero; i is in range either way
__device__ __forceinline__ double pick(const double* __restrict__ p, int i, bool ok) {
  const double x = p[i];
  return ok ? x : 0.0;
}

// out[f][a0][x1][x2] = sum_{a1,a2} w1t[a1][x1] (x + alpha y)[a0][a1][a2] w2t[a2][x2].  A wave owns 16 columns x2:
// it contracts a2 for them (KT1 tiles of 16 rows a1, in registers), then a1 for `rows` tiles of 16 rows x1.
// Waves are independent; those of other rows of the same columns repeat the first, smaller product.
template <int KT1>
__global__ __launch_bounds__(256) void k_iota_ab_f64(IotaABF64Args a, int rows) {
  const int lane = threadIdx.x & 63, j = lane & 15, h = lane >> 4;
  const int nct = (a.n2 + 15) / 16, nrt = (a.n1 + 15) / 16, ngr = (nrt + rows - 1) / rows;
  const int u = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (u >= nct * ngr) return;
  const int f = blockIdx.y / a.k0, a0 = blockIdx.y - f * a.k0;
  const int64_t slab = (int64_t)a0 * a.k1 * a.k2;
  const double* __restrict__ x = a.x[f] + slab;
  const double* __restrict__ y = a.y[f] ? a.y[f] + slab : nullptr;
  const double* __restrict__ w1t = a.w1t[f];
  const double* __restrict__ w2t = a.w2t[f];
  const double alpha = a.alpha[f];
  const int c = (u % nct) * 16 + j, cc = min(c, a.n2 - 1), rt0 = (u / nct) * rows;
  f64x4 t[KT1];
#pragma unroll
  for (int m = 0; m < KT1; ++m) t[m] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int kk = 0; kk < a.k2; kk += 4) {
    const bool ok = kk + h < a.k2;
    const int l = ok ? kk + h : 0;
    const double b = pick(w2t, l * a.n2 + cc, ok);
#pragma unroll
    for (int m = 0; m < KT1; ++m) {
      const bool in = ok && 16 * m + j < a.k1;
      const int i = in ? (16 * m + j) * a.k2 + l : 0;
      double v = x[i];
      if (y) v += alpha * y[i];
      t[m] = mma(in ? v : 0.0, b, t[m]);
    }
  }
  double* __restrict__ out = a.out + (int64_t)blockIdx.y * a.n1 * a.n2;
  const bool zero = a.zero[f];
  const int rt1 = min(nrt, rt0 + rows);
  for (int rt = rt0; rt < rt1; ++rt) {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    const int row = min(rt * 16 + j, a.n1 - 1);
#pragma unroll
    for (int m = 0; m < KT1; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = 16 * m + 4 * r + h;
        acc = mma(pick(w1t, min(k, a.k1 - 1) * a.n1 + row, k < a.k1), t[m][r], acc);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = rt * 16 + 4 * r + h;
      if (i < a.n1 && c < a.n2) out[i * a.n2 + c] = zero ? 0.0 : acc[r];
    }
  }
}

// out[f][a0][a1][a2] = beta out + alpha sum_{x1,x2} p1t[x1][a1] in[f][a0][x1][x2] p2t[x2][a2].  A workgroup owns a
// plane; its NW waves share out the tiles of 16 columns x2 and segments of the rows x1.  A wave contracts x1 for
// its columns (transposed: rows x2, columns a1), then x2 into all KT1 x KT2 tiles of the output, and the waves'
// partial tiles are summed through LDS in a fixed order.
template <int KT1, int KT2, int NW>
__global__ __launch_bounds__(64 * NW) void k_pi_ba_f64(PiBAF64Args a, int seg) {
  __shared__ double red[NW][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15, h = lane >> 4;
  const int nct = (a.n2 + 15) / 16, units = nct * ((a.n1 + seg - 1) / seg);
  const int f = blockIdx.x / a.k0, a0 = blockIdx.x - f * a.k0;
  const double* __restrict__ in = a.in + (int64_t)blockIdx.x * a.n1 * a.n2;
  f64x4 acc[KT1][KT2];
#pragma unroll
  for (int m = 0; m < KT1; ++m)
#pragma unroll
    for (int q = 0; q < KT2; ++q) acc[m][q] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int u = wave; u < units; u += NW) {
    const int x0 = (u % nct) * 16, l0 = (u / nct) * seg, l1 = min(a.n1, l0 + seg);
    const bool col = x0 + j < a.n2;
    f64x4 t[KT1];
#pragma unroll
    for (int m = 0; m < KT1; ++m) t[m] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int kk = l0; kk < l1; kk += 4) {
      const bool ok = kk + h < l1;
      const int l = ok ? kk + h : l0;
      const double v = pick(in, l * a.n2 + (col ? x0 + j : 0), ok && col);
#pragma unroll
      for (int m = 0; m < KT1; ++m) t[m] = mma(v, pick(a.p1t, l * a.k1 + min(16 * m + j, a.k1 - 1), ok), t[m]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int x2 = x0 + 4 * r + h;
#pragma unroll
      for (int q = 0; q < KT2; ++q) {
        const double b = pick(a.p2t, min(x2, a.n2 - 1) * a.k2 + min(16 * q + j, a.k2 - 1), x2 < a.n2);
#pragma unroll
        for (int m = 0; m < KT1; ++m) acc[m][q] = mma(t[m][r], b, acc[m][q]);
      }
    }
  }
  double* __restrict__ out = a.out[f] + (int64_t)a0 * a.k1 * a.k2;
  const double alpha = a.alpha[f], beta = a.beta[f];
#pragma unroll
  for (int m = 0; m < KT1; ++m)
#pragma unroll
    for (int q = 0; q < KT2; ++q) {
      if (m + q) __syncthreads();
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][r * 64 + lane] = acc[m][q][r];
      __syncthreads();
      const int tid = threadIdx.x;
      const int a1 = 16 * m + tid / 16, a2 = 16 * q + (tid & 15);
      if (tid < 256 && a1 < a.k1 && a2 < a.k2) {
        double s = red[0][tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += red[w][tid];
        const int o = a1 * a.k2 + a2;
        out[o] = beta == 0.0 ? alpha * s : beta * out[o] + alpha * s;  // beta 0 never reads out
      }
    }
}

// One axis: out[b][m][c] = sum_l A[m][l] B[l][c], a wave per 32 x 32 block of the output.  The matrix W [.][L] is A
// where a non-last axis is contracted (B = in[b], C contiguous) and, transposed, B where the last one is (A = in[b]).
template <bool LAST>
__global__ __launch_bounds__(256) void k_axis_f64(const double* __restrict__ in, double* __restrict__ out,
                                                  FieldMats<double> mats, int bpf, int M, int L, int C, int64_t sIb,
                                                  int64_t sOb) {
  const int lane = threadIdx.x & 63, j = lane & 15, h = lane >> 4;
  const int ncb = (C + 31) / 32, u = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (u >= ncb * ((M + 31) / 32)) return;
  const int b = blockIdx.y, m0 = (u / ncb) * 32, c0 = (u % ncb) * 32;
  const double* __restrict__ W = mats.w[b / bpf];
  in += b * sIb;
  out += b * sOb;
  f64x4 acc[2][2];
#pragma unroll
  for (int p = 0; p < 4; ++p) acc[p >> 1][p & 1] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int kk = 0; kk < L; kk += 4) {
    const bool ok = kk + h < L;
    const int l = ok ? kk + h : 0;
    double av[2], bv[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int64_t m = min(m0 + 16 * p + j, M - 1), c = min(c0 + 16 * p + j, C - 1);
      const double x = (LAST ? in : W)[m * L + l], y = LAST ? W[c * L + l] : in[(int64_t)l * C + c];
      av[p] = ok ? x : 0.0;
      bv[p] = ok ? y : 0.0;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) acc[p >> 1][p & 1] = mma(av[p >> 1], bv[p & 1], acc[p >> 1][p & 1]);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 16 * (p >> 1) + 4 * r + h, c = c0 + 16 * (p & 1) + j;
      if (m < M && c < C) out[(int64_t)m * C + c] = acc[p >> 1][p & 1][r];
    }
}

int ceil16(int k) { return (k + 15) / 16; }

}  // namespace

// both inner axes in one kernel: bands of up to 64 x 64 (the intermediate and the output tiles of a wave stay in
// registers) and planes that one workgroup projects in no more time than a kernel per axis over many workgroups:
// at 256 x 256 with a 64 x 64 band a call takes 99 us here, and 103 us at 300 x 300 by the axes
bool fused_f64_ok(int n1, int n2, int k1, int k2) { return k1 <= 64 && k2 <= 64 && (int64_t)n1 * n2 <= kFusedF64Plane; }

void iota_ab_f64(const IotaABF64Args& a, int nf, hipStream_t s) {
  if (!fused_f64_ok(a.n1, a.n2, a.k1, a.k2)) throw ArgError("FP64 inclusion beyond the fused kernel's range");
  const int nct = ceil16(a.n2), nrt = ceil16(a.n1);
  // a tile of rows per wave while that leaves the waves few (each repeats the first product), four beyond
  const int rows = (int64_t)nf * a.k0 * nct * nrt <= 4096 ? 1 : 4;
  const dim3 g(ceil_div(nct * ceil_div(nrt, rows), 4), nf * a.k0);
  const double P = (double)a.n1 * a.n2 * a.k0 * nf, Q = (double)a.k0 * a.k1 * a.k2 * nf;
  auto go = [&](auto* k) {
    prof::launch("k_iota_ab_f64", 8.0 * (P + Q), 2.0 * a.k1 * (Q / a.k1 * a.n2 + P), k, g, dim3(256), 0, s, a, rows);
  };
  if (a.k1 <= 16) go(k_iota_ab_f64<1>);
  else if (a.k1 <= 32) go(k_iota_ab_f64<2>);
  else go(k_iota_ab_f64<4>);
  LDDMM_LAUNCH_CHECK();
}

void pi_ba_f64(const PiBAF64Args& a, int nf, hipStream_t s) {
  if (!fused_f64_ok(a.n1, a.n2, a.k1, a.k2)) throw ArgError("FP64 projection beyond the fused kernel's range");
  const double P = (double)a.n1 * a.n2 * a.k0 * nf, Q = (double)a.k0 * a.k1 * a.k2 * nf;
  auto go = [&](auto* k, int nw) {
    // row segments so that every wave has one tile of columns (at least 16 rows: one batch of loads)
    const int parts = std::max(1, std::min(nw / ceil16(a.n2), ceil16(a.n1)));
    const int seg = ceil_div(ceil_div(a.n1, parts), 4) * 4;
    prof::launch("k_pi_ba_f64", 8.0 * (P + Q), 2.0 * a.k1 * (P + Q / a.k1 * a.n2), k, dim3(nf * a.k0), dim3(64 * nw),
                 0, s, a, seg);
  };
  const int t1 = ceil16(a.k1), t2 = ceil16(a.k2);
  if (t1 <= 1 && t2 <= 1) go(k_pi_ba_f64<1, 1, 16>, 16);
  else if (t1 <= 2 && t2 <= 2) go(k_pi_ba_f64<2, 2, 16>, 16);
  else go(k_pi_ba_f64<4, 4, 8>, 8);
  LDDMM_LAUNCH_CHECK();
}

void axis_f64(const double* in, double* out, const FieldMats<double>& W, int nb, int bpf, int M, int L, int C,
              int64_t sIb, int64_t sOb, bool last, hipStream_t s) {
  if (nb <= 0 || M <= 0 || C <= 0) return;
  if (nb > 65535) throw ArgError("axis_f64: batch too large");
  const dim3 g(ceil_div((int64_t)ceil_div(C, 32) * ceil_div(M, 32), 4), nb);
  const double bytes = 8.0 * nb * ((last ? (double)M * L : (double)L * C) + (double)M * C);
  prof::launch("k_axis_f64", bytes, 2.0 * nb * M * (double)L * C, last ? k_axis_f64<true> : k_axis_f64<false>, g,
               dim3(256), 0, s, in, out, W, bpf, M, L, C, sIb, sOb);
  LDDMM_LAUNCH_CHECK();
}

}  // namespace lddmm
