// Grid-point and band-coefficient kernels: characteristics, tricubic B-spline
// interpolation fused with the SL-RK2 step updates (Section 3), the periodic
// B-spline prefilter, source terms and products of the variants' equations
// (Sections 2.3.1, 2.3.3, Table 1) and the Jacobian determinant.
//
// Every grid kernel maps one thread to one node; fields are component-major
// [c][n0][n1][n2], n2 contiguous, so neighbouring lanes touch neighbouring nodes.
#include "kernels.h"
#include "prof.h"

#include <algorithm>
#include <type_traits>

namespace lddmm {

namespace {

constexpr int kBlock = 256;

struct GridIdx {
  int i0, i1, i2;
};

__device__ __forceinline__ GridIdx unflatten(int64_t p, int n1, int n2) {
  GridIdx g;
  g.i2 = static_cast<int>(p % n2);
  const int64_t q = p / n2;
  g.i1 = static_cast<int>(q % n1);
  g.i0 = static_cast<int>(q / n1);
  return g;
}

// Tricubic B-spline taps of one point: periodic indices and weights per axis.  A 2D problem's first axis holds one
// node, whose four taps add up to it: 16 taps instead of 64 (FP64, 64^2: an interpolation 5.1 -> 3.0 us).
template <typename T>
struct Taps {
  int i0[4], i1[4], i2[4];
  T w0[4], w1[4], w2[4];
  bool flat;
  __device__ __forceinline__ void set(T x0, T x1, T x2, int n0, int n1, int n2) {
    flat = n0 == 1;
    bspline_weights(tap_indices(x0, n0, i0), w0);
    bspline_weights(tap_indices(x1, n1, i1), w1);
    bspline_weights(tap_indices(x2, n2, i2), w2);
  }
  __device__ __forceinline__ T plane(const T* __restrict__ c, int n1, int n2, int i) const {
    T s = T(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const T* row = c + (static_cast<int64_t>(i) * n1 + i1[b]) * n2;
      const T sb = w2[0] * row[i2[0]] + w2[1] * row[i2[1]] + w2[2] * row[i2[2]] + w2[3] * row[i2[3]];
      s += w1[b] * sb;
    }
    return s;
  }
  __device__ __forceinline__ T eval(const T* __restrict__ c, int n1, int n2) const {
    if (flat) return plane(c, n1, n2, 0);
    T acc = T(0);
#pragma unroll
    for (int a = 0; a < 4; ++a) acc += w0[a] * plane(c, n1, n2, i0[a]);
    return acc;
  }
};

// ---- band coefficient kernels ----------------------------------------------

template <typename T>
__global__ void k_axpby(T* out, T a, const T* x, T b, const T* y, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  T r = a * x[i];
  if (y) r += b * y[i];
  out[i] = r;
}

template <typename T>
__global__ void k_scale_sym(T* out, const T* x, const double* sym, int ncomp, int64_t Q, const T* y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= Q * ncomp) return;
  T r = static_cast<T>(sym[i % Q]) * x[i];
  if (y) r += y[i];
  out[i] = r;
}

// derivative along one axis in the real basis: slot 2k-1 (cos) <- 2 pi k * slot 2k (sin),
// slot 2k (sin) <- -2 pi k * slot 2k-1 (cos); slot 0 and the pad slot -> 0.
__device__ __forceinline__ int deriv_src(int a, int K, double& fac) {
  const double two_pi = 6.283185307179586476925286766559;
  if (a == 0 || (K % 2 == 0 && a == K - 1)) {
    fac = 0.0;
    return a;
  }
  const int k = (a + 1) / 2;
  if (a & 1) {
    fac = two_pi * k;
    return a + 1;
  }
  fac = -two_pi * k;
  return a - 1;
}

template <typename T>
__global__ void k_bl_div(T* out, const T* v, int k0, int k1, int k2) {
  const int64_t Q = (int64_t)k0 * k1 * k2;
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= Q) return;
  const int a2 = static_cast<int>(q % k2);
  const int a1 = static_cast<int>((q / k2) % k1);
  const int a0 = static_cast<int>(q / ((int64_t)k1 * k2));
  double acc = 0.0, f;
  int s = deriv_src(a0, k0, f);
  if (k0 > 1 && f != 0.0) acc += f * static_cast<double>(v[0 * Q + ((int64_t)s * k1 + a1) * k2 + a2]);
  s = deriv_src(a1, k1, f);
  if (k1 > 1 && f != 0.0) acc += f * static_cast<double>(v[1 * Q + ((int64_t)a0 * k1 + s) * k2 + a2]);
  s = deriv_src(a2, k2, f);
  if (k2 > 1 && f != 0.0) acc += f * static_cast<double>(v[2 * Q + ((int64_t)a0 * k1 + a1) * k2 + s]);
  out[q] = static_cast<T>(acc);
}

// ---- characteristics (Section 3.1) ----------------------------------------

template <typename T>
__global__ void k_characteristics(T* __restrict__ disp, const T* __restrict__ v, const T* __restrict__ cv,
                                  int n0, int n1, int n2, T dt, int dir) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const GridIdx g = unflatten(p, n1, n2);
  const T sdt = dir > 0 ? dt : -dt;
  const T v0 = v[p] * n0, v1 = v[P + p] * n1, v2 = v[2 * P + p] * n2;  // grid units
  Taps<T> t;
  t.set(g.i0 + sdt * v0, g.i1 + sdt * v1, g.i2 + sdt * v2, n0, n1, n2);
  const T s0 = t.eval(cv, n1, n2) * n0;
  const T s1 = t.eval(cv + P, n1, n2) * n1;
  const T s2 = t.eval(cv + 2 * P, n1, n2) * n2;
  const T h = T(0.5) * sdt;
  disp[p] = h * (v0 + s0);
  disp[P + p] = h * (v1 + s1);
  disp[2 * P + p] = h * (v2 + s2);
}

template <typename T, int NF>
__global__ void k_interp(T* __restrict__ out, const T* __restrict__ c, const T* __restrict__ disp, int n0,
                         int n1, int n2) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const GridIdx g = unflatten(p, n1, n2);
  Taps<T> t;
  t.set(g.i0 + disp[p], g.i1 + disp[P + p], g.i2 + disp[2 * P + p], n0, n1, n2);
#pragma unroll
  for (int f = 0; f < NF; ++f) out[f * P + p] = t.eval(c + f * P, n1, n2);
}

// variant-1 adjoint (Table 1 row 2, -D_t lambda = lambda div v), one Heun step
template <typename T>
__global__ void k_adjoint_grid_step(T* __restrict__ out, const T* __restrict__ c1, const T* __restrict__ c2,
                                    const T* __restrict__ disp, const T* __restrict__ divv, int n0, int n1, int n2,
                                    T dt) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const GridIdx g = unflatten(p, n1, n2);
  Taps<T> t;
  t.set(g.i0 + disp[p], g.i1 + disp[P + p], g.i2 + disp[2 * P + p], n0, n1, n2);
  const T a = t.eval(c1, n1, n2), b = t.eval(c2, n1, n2);
  out[p] = a + T(0.5) * dt * (b + (a + dt * b) * divv[p]);
}

// band-limited adjoint step: out_f = cA_f o X + dt/2 divv (cB_f o X)
template <typename T, int NF>
__global__ void k_bl_adjoint_step(T* __restrict__ out, const T* __restrict__ cA, const T* __restrict__ cB,
                                  const T* __restrict__ disp, const T* __restrict__ divv, int n0, int n1, int n2,
                                  T dt) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const GridIdx g = unflatten(p, n1, n2);
  Taps<T> t;
  t.set(g.i0 + disp[p], g.i1 + disp[P + p], g.i2 + disp[2 * P + p], n0, n1, n2);
  const T hd = T(0.5) * dt * divv[p];
#pragma unroll
  for (int f = 0; f < NF; ++f) out[f * P + p] = t.eval(cA + f * P, n1, n2) + hd * t.eval(cB + f * P, n1, n2);
}

template <typename T>
__device__ __forceinline__ void v3_src_point(T o[3], const T* __restrict__ Du, const T* __restrict__ dv,
                                             int64_t p, int64_t P) {
  const T w0 = dv[p], w1 = dv[P + p], w2 = dv[2 * P + p];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const T* D = Du + (int64_t)(3 * i) * P;  // d_j u_i at D[j * P]
    o[i] = (i == 0 ? w0 : (i == 1 ? w1 : w2)) - (D[p] * w0 + D[P + p] * w1 + D[2 * P + p] * w2);
  }
}

template <typename T>
__global__ void k_v3_source(T* __restrict__ out, const T* __restrict__ Du, const T* __restrict__ dv, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  T o[3];
  v3_src_point(o, Du, dv, p, P);
  out[p] = o[0];
  out[P + p] = o[1];
  out[2 * P + p] = o[2];
}

template <typename T>
__global__ void k_v1_source(T* __restrict__ out, const T* __restrict__ G, const T* __restrict__ dv, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  out[p] = -(G[p] * dv[p] + G[P + p] * dv[P + p] + G[2 * P + p] * dv[2 * P + p]);
}

template <typename T>
__global__ void k_v1_products(T* __restrict__ out, const T* __restrict__ e, const T* __restrict__ divv,
                              const T* __restrict__ G, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const T x = e[p];
  out[p] = x * divv[p];
  out[P + p] = x * G[p];
  out[2 * P + p] = x * G[P + p];
  out[3 * P + p] = x * G[2 * P + p];
}

template <typename T>
__global__ void k_v3_products(T* __restrict__ out, const T* __restrict__ e, const T* __restrict__ divv,
                              const T* __restrict__ Du, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const T r0 = e[p], r1 = e[P + p], r2 = e[2 * P + p], dv = divv[p];
  out[p] = r0 * dv;
  out[P + p] = r1 * dv;
  out[2 * P + p] = r2 * dv;
  // (Du)^T r: component j = sum_i r_i d_j u_i, Du[(3 i + j) P]
#pragma unroll
  for (int j = 0; j < 3; ++j)
    out[(3 + j) * P + p] = r0 * Du[(0 + j) * P + p] + r1 * Du[(3 + j) * P + p] + r2 * Du[(6 + j) * P + p];
}

// Transformation of a grid field through per-node maps (state-equation variant, Section 2.3.2):
// out_n(x) = a w_n(x) P(c)(x - u_n(x)), n = blockIdx.y, with u_n a displacement in unit-torus units
// ([n][3][P]) and w_n an optional weight field ([n][P]).  One gather of the 64 taps per node: the
// displacements here are whole deformations, not one step's, so no brick around the node holds them.
template <typename T>
__global__ void k_pull_back(T* __restrict__ out, const T* __restrict__ c, const T* __restrict__ u,
                            const T* __restrict__ w, T a, int n0, int n1, int n2) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const int64_t node = blockIdx.y;
  const T* un = u + node * 3 * P;
  const GridIdx g = unflatten(p, n1, n2);
  Taps<T> t;
  t.set(g.i0 - un[p] * n0, g.i1 - un[P + p] * n1, g.i2 - un[2 * P + p] * n2, n0, n1, n2);
  T r = a * t.eval(c, n1, n2);
  if (w) r *= w[node * P + p];
  out[node * P + p] = r;
}

// out_j = sum_n e_n G_n,j (e [ns][P], G [ns][3][P]): the time integral of the state-equation variant's
// gradient and Hessian terms on the product grid, its weights folded into e_n
template <typename T>
__global__ void k_node_sum(T* __restrict__ out, const T* __restrict__ e, const T* __restrict__ G, int ns, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  T a0 = 0, a1 = 0, a2 = 0;
  for (int n = 0; n < ns; ++n) {
    const T x = e[n * P + p];
    const T* g = G + 3 * n * P;
    a0 += x * g[p];
    a1 += x * g[P + p];
    a2 += x * g[2 * P + p];
  }
  out[p] = a0;
  out[P + p] = a1;
  out[2 * P + p] = a2;
}

// Right-hand sides of the explicit RK comparator (deformation-state equations in Eulerian form) on the
// product grid, where the truncated products are exact:
//   adjoint:            out_i = -(sum_j d_j r_i v_j + r_i div v)   (the product rule of -div(r_i v))
//   incremental state:  out_i = dv_i - sum_j d_j du_i v_j - sum_j (a Du_a + b Du_b)_ij dv_j
// (D fields [i][j] = d_j x_i, 9 per vector)
template <typename T>
__global__ void k_rk_adjoint_rhs(T* __restrict__ out, const T* __restrict__ Dr, const T* __restrict__ r,
                                 const T* __restrict__ v, const T* __restrict__ divv, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const T v0 = v[p], v1 = v[P + p], v2 = v[2 * P + p], dv = divv[p];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const T* D = Dr + 3 * i * P;
    out[i * P + p] = -(D[p] * v0 + D[P + p] * v1 + D[2 * P + p] * v2 + r[i * P + p] * dv);
  }
}

template <typename T>
__global__ void k_rk_inc_rhs(T* __restrict__ out, const T* __restrict__ Ddu, const T* __restrict__ Dua,
                             const T* __restrict__ Dub, T a, T b, const T* __restrict__ v, const T* __restrict__ dv,
                             int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const T v0 = v[p], v1 = v[P + p], v2 = v[2 * P + p];
  const T w0 = dv[p], w1 = dv[P + p], w2 = dv[2 * P + p];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const T* D = Ddu + 3 * i * P;
    const T* A = Dua + 3 * i * P;
    const T* B = Dub + 3 * i * P;
    const T u0 = a * A[p] + b * B[p], u1 = a * A[P + p] + b * B[P + p], u2 = a * A[2 * P + p] + b * B[2 * P + p];
    out[i * P + p] = dv[i * P + p] - (D[p] * v0 + D[P + p] * v1 + D[2 * P + p] * v2) - (u0 * w0 + u1 * w1 + u2 * w2);
  }
}

template <typename T>
__global__ void k_band_copy(T* __restrict__ out, int o0, int o1, int o2, const T* __restrict__ in, int i0, int i1,
                            int i2, int m0, int m1, int m2, int ncomp, bool keep_rest) {
  const int64_t Qo = (int64_t)o0 * o1 * o2;
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= ncomp * Qo) return;
  const int c = static_cast<int>(q / Qo);
  const int64_t r = q - c * Qo;
  const int a2 = static_cast<int>(r % o2), a1 = static_cast<int>((r / o2) % o1), a0 = static_cast<int>(r / ((int64_t)o1 * o2));
  if (a0 < m0 && a1 < m1 && a2 < m2)
    out[q] = in[(int64_t)c * i0 * i1 * i2 + ((int64_t)a0 * i1 + a1) * i2 + a2];
  else if (!keep_rest)
    out[q] = T(0);
}

template <typename T>
__global__ void k_restrict_grid(T* __restrict__ out, const T* __restrict__ in, int n0, int n1, int n2, int f0,
                                int f1, int f2) {
  const int c0 = n0 / f0, c1 = n1 / f1, c2 = n2 / f2;
  const int64_t Pc = (int64_t)c0 * c1 * c2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= Pc) return;
  const GridIdx g = unflatten(p, c1, c2);
  T acc = 0;
  for (int a = 0; a < f0; ++a)
    for (int b = 0; b < f1; ++b)
      for (int e = 0; e < f2; ++e)
        acc += in[((int64_t)(g.i0 * f0 + a) * n1 + (g.i1 * f1 + b)) * n2 + (g.i2 * f2 + e)];
  out[p] = acc / T(f0 * f1 * f2);
}

template <typename T>
__global__ void k_final_warp(T* __restrict__ m1, T* __restrict__ g1, const T* __restrict__ cI0,
                             const T* __restrict__ u, int n0, int n1, int n2) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const GridIdx g = unflatten(p, n1, n2);
  int i0[4], i1[4], i2[4];
  T w0[4], w1[4], w2[4], d0[4], d1[4], d2[4];
  const T t0 = tap_indices(g.i0 - u[p] * n0, n0, i0);
  const T t1 = tap_indices(g.i1 - u[P + p] * n1, n1, i1);
  const T t2 = tap_indices(g.i2 - u[2 * P + p] * n2, n2, i2);
  bspline_weights(t0, w0);
  bspline_weights(t1, w1);
  bspline_weights(t2, w2);
  bspline_dweights(t0, d0);
  bspline_dweights(t1, d1);
  bspline_dweights(t2, d2);
  T val = 0, gx = 0, gy = 0, gz = 0;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    T sv = 0, sy = 0, sz = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const T* row = cI0 + (static_cast<int64_t>(i0[a]) * n1 + i1[b]) * n2;
      const T r0 = row[i2[0]], r1 = row[i2[1]], r2 = row[i2[2]], r3 = row[i2[3]];
      const T s = w2[0] * r0 + w2[1] * r1 + w2[2] * r2 + w2[3] * r3;
      const T sd = d2[0] * r0 + d2[1] * r1 + d2[2] * r2 + d2[3] * r3;
      sv += w1[b] * s;
      sy += d1[b] * s;
      sz += w1[b] * sd;
    }
    val += w0[a] * sv;
    gx += d0[a] * sv;
    gy += w0[a] * sy;
    gz += w0[a] * sz;
  }
  m1[p] = val;
  g1[p] = gx * n0;
  g1[P + p] = gy * n1;
  g1[2 * P + p] = gz * n2;
}

template <typename T>
__global__ void k_scaled_diff(T* out, T a, const T* x, const T* y, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = a * (x[i] - y[i]);
}

template <typename T>
__global__ void k_residual_times_grad(T* out, T a, const T* x, const T* y, const T* g1, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const T r = a * (x[p] - y[p]);
  out[p] = r * g1[p];
  out[P + p] = r * g1[P + p];
  out[2 * P + p] = r * g1[2 * P + p];
}

template <typename T>
__global__ void k_coupling_v3(T* out, T a, const T* g1, const T* w, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const T s = a * (g1[p] * w[p] + g1[P + p] * w[P + p] + g1[2 * P + p] * w[2 * P + p]);
  out[p] = s * g1[p];
  out[P + p] = s * g1[P + p];
  out[2 * P + p] = s * g1[2 * P + p];
}

template <typename T>
__global__ void k_mul(T* out, const T* x, const T* y, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = x[i] * y[i];
}

template <typename T>
__global__ void k_copy(T* __restrict__ dst, const T* __restrict__ src, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

template <typename T>
__global__ void k_zero(T* p, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = T(0);
}

template <typename T>
__global__ void k_jacobian(double* out, const T* Du, int64_t P) {
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  double A[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) A[i][j] = (i == j ? 1.0 : 0.0) - static_cast<double>(Du[(3 * i + j) * P + p]);
  out[p] = A[0][0] * (A[1][1] * A[2][2] - A[1][2] * A[2][1]) - A[0][1] * (A[1][0] * A[2][2] - A[1][2] * A[2][0]) +
           A[0][2] * (A[1][0] * A[2][1] - A[1][1] * A[2][0]);
}

// ---- periodic cubic B-spline prefilter -----------------------------------------
// Interpolating coefficients c of samples f solve (c[i-1] + 4 c[i] + c[i+1]) / 6 = f[i]
// on a periodic line.  The inverse filter factors into a causal and an anti-causal
// first-order recursion with pole z = sqrt(3) - 2 and gain 6; the periodic start
// values are the geometrically weighted wrap-around sums (truncated where z^h is
// below the working precision).
//
// One pass per axis, out of place.  A thread filters a chunk of 16 points of a line: it requests the chunk
// and the points around it that the two recursions still feel (W before, W after) at once, runs the causal
// recursion from zero through the points before, and the anti-causal one from zero through those after, in
// registers and in double.  Chunks are independent, so nothing is staged, no thread waits for another, and a
// pass is a few microseconds of load latency: 128^3, one field 15.8 -> 7.5 us per axis (16.8 MB at 2.2 TB/s; the
// neighbours' points come from the caches), two fields 11.2, against a staged tile of lines whose serial start
// sums and recursions each waited for LDS.  FP64 64^2: 7.7 -> 7.4 us (a 2D field of this size takes the kernel below).
template <typename T>
struct Pole {
  static constexpr double z = -0.26794919243112270647255365849413;  // sqrt(3) - 2
  static constexpr int W = sizeof(T) == 4 ? 16 : 32;                // |z|^W below the working precision
};
constexpr int kChunk = 16;
constexpr int kMaxPrefilter = 2;  // fields of one call

template <typename T>
struct PrefilterArgs {
  const T* src[kMaxPrefilter];
  const T* w[kMaxPrefilter];  // optional pointwise factor of the samples
  T* dst;
  int n;           // points of a line
  int64_t stride;  // between points of a line
  int64_t inner, outer_stride;  // lines: inner consecutive ones at stride 1, repeated at outer_stride (ROWS: inner rows)
  int outer;
  int64_t P;
};

// ROWS: lines along the contiguous axis, lanes on consecutive chunks (VEC: rows of a multiple of four points,
// read as 16-byte quads).  Otherwise lanes on consecutive lines, the points' addresses uniform.  The index
// advances by compare and select (a wrapped index per point, inlined, made the code 23 KB and the pass
// bound by fetching it).
template <typename T, bool ROWS, bool VEC>
__global__ __launch_bounds__(256) void k_prefilter(PrefilterArgs<T> a) {
  constexpr int C = kChunk, W = Pole<T>::W, N = C + 2 * W, STEP = VEC ? 4 : 1;
  typedef T T4 __attribute__((ext_vector_type(4)));
  const int n = a.n;
  int field, c0;
  int64_t line;    // first point of the line (ROWS), or of the lines' row of points
  unsigned q = 0;  // the lane's line among consecutive ones
  if constexpr (ROWS) {
    const int nch = (n + C - 1) / C;
    const int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (t >= a.inner * nch) return;
    field = blockIdx.y;
    line = (t / nch) * n;
    c0 = (int)(t % nch) * C;
  } else {
    q = blockIdx.x * 64u + (threadIdx.x & 63);
    c0 = __builtin_amdgcn_readfirstlane(blockIdx.y * 4 + (threadIdx.x >> 6)) * C;
    if (q >= a.inner || c0 >= n) return;
    field = blockIdx.z / a.outer;
    line = (blockIdx.z - field * a.outer) * a.outer_stride;
  }
  int first = c0 - W;  // periodic index of the first point felt
  first = (first % n + n) % n;
  T v[N];
  auto fetch = [&](const T* __restrict__ f, auto&& use) {
    int i = first;
#pragma unroll
    for (int k = 0; k < N; k += STEP) {
      if constexpr (VEC) {
        const T4 x = *reinterpret_cast<const T4*>(f + line + i);
#pragma unroll
        for (int j = 0; j < 4; ++j) use(v[k + j], x[j]);
      } else if constexpr (ROWS) {
        use(v[k], f[line + i]);
      } else {
        const T* p = f + line + i * a.stride;
        use(v[k], p[q]);
      }
      i = i + STEP >= n ? 0 : i + STEP;
    }
  };
  fetch(a.src[field], [](T& d, T x) { d = x; });
  if (a.w[field]) fetch(a.w[field], [](T& d, T x) { d *= x; });
  // causal: y[i] = f[i] + z y[i-1]; anti-causal: u[i] = y[i] + z u[i+1]; c = -6 z u
  const double z = Pole<T>::z;
  double y[C + W], prev = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) prev = fma(z, prev, static_cast<double>(v[k]));
#pragma unroll
  for (int k = 0; k < C + W; ++k) y[k] = prev = fma(z, prev, static_cast<double>(v[W + k]));
  prev = 0.0;
#pragma unroll
  for (int k = C + W - 1; k >= C; --k) prev = fma(z, prev, y[k]);
#pragma unroll
  for (int k = C - 1; k >= 0; --k) {
    prev = fma(z, prev, y[k]);
    y[k] = -6.0 * z * prev;
  }
  T* __restrict__ dst = a.dst + field * a.P + line;
  if constexpr (VEC) {
#pragma unroll
    for (int k = 0; k < C; k += 4) {
      T4 x;
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = static_cast<T>(y[k + j]);
      if (c0 + k < n) *reinterpret_cast<T4*>(dst + c0 + k) = x;
    }
  } else {
#pragma unroll
    for (int k = 0; k < C; ++k)
      if (c0 + k < n) {
        T* p = dst + (ROWS ? (int64_t)(c0 + k) : (c0 + k) * a.stride);
        p[q] = static_cast<T>(y[k]);
      }
  }
}

// Both inner axes of a plane in one workgroup: the plane is staged once (rows of an odd pitch, so lanes on
// consecutive rows meet different banks), each thread filters one chunk of either axis straight from LDS as above.
// A 2D field of a few thousand nodes is then one launch instead of two (FP64 64^2: 13.5 -> 6.4 us), a 3D one two
// instead of three, of 80 KB and a chunk of 64 lines per wave at most (one workgroup a CU; 128^3, two fields: 34 -> 24 us, one 22 -> 17.5).
constexpr int kPlaneThreads = 1024;
constexpr int kPlaneBytes = 81920;

// TILE: a workgroup takes 64 columns of a plane (blockIdx.z) with the W columns on either side that their recursions
// along the rows still feel, so twice the workgroups share 128^2 planes and planes of more columns fit.
constexpr int kPlaneTile = 64;

template <typename T, bool TILE, int NT, int BYTES>
__global__ __launch_bounds__(NT) void k_prefilter_plane(PrefilterArgs<T> a, int n1, int n2) {
  constexpr int C = kChunk, W = Pole<T>::W, OFF = TILE ? W : 0;
  __shared__ T s[BYTES / sizeof(T)];
  const int tid = threadIdx.x, field = blockIdx.y;
  const int x0 = TILE ? blockIdx.z * kPlaneTile : 0, cols = TILE ? min(kPlaneTile, n2 - x0) : n2;
  const int width = TILE ? kPlaneTile + 2 * W : n2, pitch = width | 1;
  const int64_t plane = (int64_t)blockIdx.x * n1 * n2;
  const T* __restrict__ f = a.src[field] + plane;
  const T* __restrict__ w = a.w[field] ? a.w[field] + plane : nullptr;
  {
    constexpr int U = 8;  // values requested together
    const int dr = NT / width, dc = NT - dr * width, total = n1 * width;
    int r = tid / width, c = tid - r * width;
    for (int p0 = tid; p0 < total; p0 += NT * U) {
      T v[U], u[U];
      int at[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const bool ok = p0 + NT * k < total;
        int col = c + x0 - OFF;
        if (TILE) col = col < 0 ? col + n2 : col >= n2 ? col - n2 : col;
        const int p = ok ? r * n2 + col : 0;
        at[k] = ok ? r * pitch + c : -1;
        v[k] = f[p];
        if (w) u[k] = w[p];
        r += dr, c += dc;
        if (c >= width) c -= width, ++r;
      }
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (at[k] >= 0) s[at[k]] = w ? v[k] * u[k] : v[k];
    }
  }
  // lines of n points at distance `step`, line l at l * across: a wave filters one chunk of 64 lines (the wrapped
  // index is uniform: in vector registers its compare and select cost more than the recursions)
  // (a tile's rows hold their halo and do not wrap)
  auto pass = [&](int n, bool wrap, const T* base, int step, int lines, int across, auto&& put) {
    const int groups = (lines + 63) / 64, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = wave % groups * 64 + (tid & 63), c0 = wave / groups * C;
    const bool mine = c0 < n && l < lines;
    double y[C + W];
    __syncthreads();
    if (mine) {
      const T* line = base + l * across;
      int i = c0 - W;
      if (wrap) i %= n, i = i < 0 ? i + n : i;
      auto next = [&] {
        const double x = static_cast<double>(line[i * step]);
        ++i;
        if (wrap && i == n) i = 0;
        return x;
      };
      const double z = Pole<T>::z;
      double prev = 0.0;
#pragma unroll 8
      for (int k = 0; k < W; ++k) prev = fma(z, prev, next());
#pragma unroll
      for (int k = 0; k < C + W; ++k) y[k] = prev = fma(z, prev, next());
      prev = 0.0;
#pragma unroll
      for (int k = C + W - 1; k >= C; --k) prev = fma(z, prev, y[k]);
#pragma unroll
      for (int k = C - 1; k >= 0; --k) {
        prev = fma(z, prev, y[k]);
        y[k] = -6.0 * z * prev;
      }
    }
    put(mine, l, c0, y);
  };
  T* __restrict__ dst = a.dst + field * a.P + plane;
  pass(cols, !TILE, s + OFF, 1, n1, pitch, [&](bool ok, int l, int c0, const double (&y)[C + W]) {
    __syncthreads();
    if (ok)
#pragma unroll
      for (int k = 0; k < C; ++k)
        if (c0 + k < cols) s[l * pitch + OFF + c0 + k] = static_cast<T>(y[k]);
  });
  pass(n1, true, s + OFF, pitch, cols, 1, [&](bool ok, int l, int c0, const double (&y)[C + W]) {
    if (ok)
#pragma unroll
      for (int k = 0; k < C; ++k)
        if (c0 + k < n1) dst[(c0 + k) * n2 + x0 + l] = static_cast<T>(y[k]);
  });
}

inline dim3 grid_for(int64_t n) { return dim3(ceil_div(n, kBlock)); }

}  // namespace

// ---- launchers -----------------------------------------------------------------

template <typename T>
void bl_axpby(T* out, T a, const T* x, T b, const T* y, int64_t n, hipStream_t s) {
  prof::launch(std::string("k_axpby<") + prof::tname<T>() + ">", (y ? 3.0 : 2.0) * n * sizeof(T), 0.0, k_axpby<T>, grid_for(n), dim3(kBlock), 0, s, out, a, x, b, y, n);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void bl_scale_sym(T* out, const T* x, const double* sym, int ncomp, int64_t Q, const T* y, hipStream_t s) {
  prof::launch(std::string("k_scale_sym<") + prof::tname<T>() + ">", 3.0 * Q * ncomp * sizeof(T), 0.0, k_scale_sym<T>, grid_for(Q * ncomp), dim3(kBlock), 0, s, out, x, sym, ncomp, Q, y);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void bl_div(T* out, const T* v, const Dims& d, hipStream_t s) {
  prof::launch(std::string("k_bl_div<") + prof::tname<T>() + ">", 4.0 * d.Q * sizeof(T), 0.0, k_bl_div<T>, grid_for(d.Q), dim3(kBlock), 0, s, out, v, d.k[0], d.k[1], d.k[2]);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void characteristics(T* disp, const T* v, const T* cv, const Dims& d, T dt, int dir, hipStream_t s) {
  if constexpr (std::is_same_v<T, float>) {
    if (brick_ok(d)) return brick_characteristics(disp, v, cv, d, dt, dir, s);
  }
  prof::launch("k_characteristics<" + std::string(prof::tname<T>()) + ">", 9.0 * d.P * sizeof(T), 0.0, k_characteristics<T>, grid_for(d.P), dim3(kBlock), 0, s, disp, v, cv, d.n[0], d.n[1], d.n[2], dt, dir);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void interp(T* out, const T* coef, int nf, const T* disp, const Dims& d, hipStream_t s) {
  if constexpr (std::is_same_v<T, float>) {
    if (brick_ok(d) && (nf == 1 || nf == 3)) return brick_interp(out, coef, nf, disp, d, s);
  }
  switch (nf) {
    case 1:
      prof::launch("k_interp<" + std::string(prof::tname<T>()) + "," + std::to_string(nf) + ">", (3.0 + 2.0 * nf) * d.P * sizeof(T), 0.0, k_interp<T, 1>, grid_for(d.P), dim3(kBlock), 0, s, out, coef, disp, d.n[0], d.n[1], d.n[2]);
      break;
    case 2:
      prof::launch("k_interp<" + std::string(prof::tname<T>()) + "," + std::to_string(nf) + ">", (3.0 + 2.0 * nf) * d.P * sizeof(T), 0.0, k_interp<T, 2>, grid_for(d.P), dim3(kBlock), 0, s, out, coef, disp, d.n[0], d.n[1], d.n[2]);
      break;
    case 3:
      prof::launch("k_interp<" + std::string(prof::tname<T>()) + "," + std::to_string(nf) + ">", (3.0 + 2.0 * nf) * d.P * sizeof(T), 0.0, k_interp<T, 3>, grid_for(d.P), dim3(kBlock), 0, s, out, coef, disp, d.n[0], d.n[1], d.n[2]);
      break;
    default:
      throw ArgError("interp: nf must be 1..3");
  }
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void prefilter(T* dst, T* tmp, const T* const* src, const T* const* w, int nf, const Dims& d, hipStream_t s) {
  if (nf < 1 || nf > kMaxPrefilter) throw ArgError("prefilter: 1 or 2 fields");
  const int n0 = d.n[0], n1 = d.n[1], n2 = d.n[2];
  int left = (n0 > 1) + (n1 > 1) + (n2 > 1);
  const std::string nm = std::string("k_prefilter<") + prof::tname<T>() + ">";
  PrefilterArgs<T> a{};
  for (int f = 0; f < nf; ++f) a.src[f] = src[f], a.w[f] = w ? w[f] : nullptr;
  a.P = d.P;
  // passes alternate between dst and tmp so that the last one writes dst
  auto pass = [&](int axis) {
    --left;
    a.dst = (left & 1) ? tmp : dst;
    a.n = d.n[axis];
    const double bytes = 2.0 * nf * d.P * sizeof(T);
    const int nch = ceil_div(a.n, kChunk);
    if (axis == 2) {
      a.stride = 1, a.inner = (int64_t)n0 * n1, a.outer = 1, a.outer_stride = 0;
      const dim3 g(ceil_div(a.inner * nch, 256), nf);
      if (n2 % 4 == 0) prof::launch(nm, bytes, 0.0, k_prefilter<T, true, true>, g, dim3(256), 0, s, a);
      else prof::launch(nm, bytes, 0.0, k_prefilter<T, true, false>, g, dim3(256), 0, s, a);
    } else {
      a.stride = axis == 1 ? n2 : (int64_t)n1 * n2;
      a.inner = a.stride;
      a.outer = axis == 1 ? n0 : 1;
      a.outer_stride = (int64_t)n1 * n2;
      const dim3 g(ceil_div(a.inner, 64), ceil_div(nch, 4), a.outer * nf);
      prof::launch(nm, bytes, 0.0, k_prefilter<T, false, false>, g, dim3(256), 0, s, a);
    }
    LDDMM_LAUNCH_CHECK();
    for (int f = 0; f < nf; ++f) a.src[f] = a.dst + f * d.P, a.w[f] = nullptr;
  };
  if (left == 0)  // a single point: its own coefficient
    for (int f = 0; f < nf; ++f) {
      if (a.w[f]) mul<T>(dst + f * d.P, a.src[f], a.w[f], d.P, s);
      else copy_dev<T>(dst + f * d.P, a.src[f], d.P, s);
    }
  constexpr int W = Pole<T>::W, kWide = (kPlaneTile + 2 * W) | 1;
  // LDS and waves of whole planes, or of 64 columns of one: tiles where a plane does not fit, or the planes leave CUs
  // idle (128^3, one field 12.9 -> 10.5 us; two, whose planes do not, 14.6 against 15.8 in tiles)
  auto lds_of = [&](bool t) { return (int64_t)n1 * (t ? kWide : n2 | 1) * (int64_t)sizeof(T); };
  auto waves_of = [&](bool t) {
    return std::max((t ? kPlaneTile / kChunk : ceil_div(n2, kChunk)) * ceil_div(n1, 64),
                    ceil_div(n1, kChunk) * (t ? 1 : ceil_div(n2, 64)));
  };
  auto fits = [&](bool t) { return lds_of(t) <= kPlaneBytes && waves_of(t) <= kPlaneThreads / 64; };
  const bool tile = n2 >= kPlaneTile + 2 * W && ((int64_t)n0 * nf < 256 || !fits(false));  // (a halo wraps once)
  const int64_t lds = lds_of(tile);
  const int waves = waves_of(tile);
  if (n1 > 1 && n2 > 1 && fits(tile)) {
    left = n0 > 1;
    a.dst = left ? tmp : dst;
    auto go = [&](auto* k, int nt) {
      prof::launch(nm, 2.0 * nf * d.P * sizeof(T), 0.0, k, dim3(n0, nf, tile ? ceil_div(n2, kPlaneTile) : 1), dim3(nt), 0,
                   s, a, n1, n2);
    };
    if (!tile) go(k_prefilter_plane<T, false, 1024, kPlaneBytes>, 1024);
    else if (waves <= 8 && lds <= 53248) go(k_prefilter_plane<T, true, 512, 53248>, 512);
    else go(k_prefilter_plane<T, true, 1024, kPlaneBytes>, 1024);
    LDDMM_LAUNCH_CHECK();
    for (int f = 0; f < nf; ++f) a.src[f] = a.dst + f * d.P, a.w[f] = nullptr;
    if (n0 > 1) pass(0);
    return;
  }
  for (int axis = 2; axis >= 0; --axis)
    if (d.n[axis] > 1) pass(axis);
}

template <typename T>
void adjoint_grid_step(T* out, const T* c1, const T* c2, const T* disp, const T* divv, const Dims& d, T dt,
                       hipStream_t s) {
  if constexpr (std::is_same_v<T, float>) {
    if (brick_ok(d) && c2 == c1 + d.P) return brick_adjoint_grid_step(out, c1, disp, divv, d, dt, s);
  }
  prof::launch("k_adjoint_grid_step<" + std::string(prof::tname<T>()) + ">", 7.0 * d.P * sizeof(T), 0.0, k_adjoint_grid_step<T>, grid_for(d.P), dim3(kBlock), 0, s, out, c1, c2, disp, divv, d.n[0], d.n[1], d.n[2], dt);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void bl_adjoint_step(T* out, const T* cA, const T* cB, int nf, const T* disp, const T* divv, const Dims& d, T dt,
                     hipStream_t s) {
  if constexpr (std::is_same_v<T, float>) {
    if (brick_ok(d) && cB == cA + nf * d.P) return brick_bl_adjoint_step(out, cA, nf, disp, divv, d, dt, s);
  }
  if (nf == 1)
    prof::launch("k_bl_adjoint_step<" + std::string(prof::tname<T>()) + "," + std::to_string(nf) + ">", (4.0 + 3.0 * nf) * d.P * sizeof(T), 0.0, k_bl_adjoint_step<T, 1>, grid_for(d.P), dim3(kBlock), 0, s, out, cA, cB, disp, divv, d.n[0], d.n[1], d.n[2], dt);
  else if (nf == 3)
    prof::launch("k_bl_adjoint_step<" + std::string(prof::tname<T>()) + "," + std::to_string(nf) + ">", (4.0 + 3.0 * nf) * d.P * sizeof(T), 0.0, k_bl_adjoint_step<T, 3>, grid_for(d.P), dim3(kBlock), 0, s, out, cA, cB, disp, divv, d.n[0], d.n[1], d.n[2], dt);
  else
    throw ArgError("bl_adjoint_step: nf must be 1 or 3");
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void v3_source(T* out, const T* Du, const T* dv, const Dims& d, hipStream_t s) {
  prof::launch("k_v3_source<" + std::string(prof::tname<T>()) + ">", 15.0 * d.P * sizeof(T), 0.0, k_v3_source<T>, grid_for(d.P), dim3(kBlock), 0, s, out, Du, dv, d.P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void v1_source(T* out, const T* G, const T* dv, const Dims& d, hipStream_t s) {
  prof::launch("k_v1_source<" + std::string(prof::tname<T>()) + ">", 7.0 * d.P * sizeof(T), 0.0, k_v1_source<T>, grid_for(d.P), dim3(kBlock), 0, s, out, G, dv, d.P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void v1_products(T* out, const T* e, const T* divv, const T* G, const Dims& d, hipStream_t s) {
  prof::launch("k_v1_products<" + std::string(prof::tname<T>()) + ">", 9.0 * d.P * sizeof(T), 0.0, k_v1_products<T>, grid_for(d.P), dim3(kBlock), 0, s, out, e, divv, G, d.P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void v3_products(T* out, const T* e, const T* divv, const T* Du, const Dims& d, hipStream_t s) {
  prof::launch("k_v3_products<" + std::string(prof::tname<T>()) + ">", 19.0 * d.P * sizeof(T), 0.0, k_v3_products<T>, grid_for(d.P), dim3(kBlock), 0, s, out, e, divv, Du, d.P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void final_warp(T* m1, T* g1, const T* cI0, const T* u, const Dims& d, hipStream_t s) {
  prof::launch("k_final_warp<" + std::string(prof::tname<T>()) + ">", 8.0 * d.P * sizeof(T), 0.0, k_final_warp<T>, grid_for(d.P), dim3(kBlock), 0, s, m1, g1, cI0, u, d.n[0], d.n[1], d.n[2]);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void pull_back(T* out, const T* c, const T* u, const T* w, T a, int nodes, const Dims& d, hipStream_t s) {
  if (nodes < 1 || nodes > 65535) throw ArgError("pull_back: node count out of range");
  const dim3 g(static_cast<unsigned>((d.P + kBlock - 1) / kBlock), static_cast<unsigned>(nodes));
  prof::launch("k_pull_back<" + std::string(prof::tname<T>()) + ">",
               double(nodes) * (w ? 5.0 : 4.0) * d.P * sizeof(T) + d.P * sizeof(T), 0.0, k_pull_back<T>, g,
               dim3(kBlock), 0, s, out, c, u, w, a, d.n[0], d.n[1], d.n[2]);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void node_sum(T* out, const T* e, const T* G, int ns, int64_t P, hipStream_t s) {
  prof::launch("k_node_sum<" + std::string(prof::tname<T>()) + ">", (4.0 * ns + 3.0) * P * sizeof(T), 0.0,
               k_node_sum<T>, grid_for(P), dim3(kBlock), 0, s, out, e, G, ns, P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void rk_adjoint_rhs(T* out, const T* Dr, const T* r, const T* v, const T* divv, int64_t P, hipStream_t s) {
  prof::launch("k_rk_adjoint_rhs<" + std::string(prof::tname<T>()) + ">", 20.0 * P * sizeof(T), 0.0,
               k_rk_adjoint_rhs<T>, grid_for(P), dim3(kBlock), 0, s, out, Dr, r, v, divv, P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void rk_inc_rhs(T* out, const T* Ddu, const T* Dua, const T* Dub, T a, T b, const T* v, const T* dv, int64_t P,
                hipStream_t s) {
  prof::launch("k_rk_inc_rhs<" + std::string(prof::tname<T>()) + ">", 39.0 * P * sizeof(T), 0.0, k_rk_inc_rhs<T>,
               grid_for(P), dim3(kBlock), 0, s, out, Ddu, Dua, Dub, a, b, v, dv, P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void band_copy(T* out, const int ko[3], const T* in, const int ki[3], const int m[3], int ncomp, bool keep_rest,
               hipStream_t s) {
  const int64_t n = (int64_t)ncomp * ko[0] * ko[1] * ko[2];
  for (int j = 0; j < 3; ++j)
    if (m[j] > ko[j] || m[j] > ki[j]) throw ArgError("band_copy: copy extent beyond a band");
  prof::launch("k_band_copy<" + std::string(prof::tname<T>()) + ">", 2.0 * n * sizeof(T), 0.0, k_band_copy<T>,
               grid_for(n), dim3(kBlock), 0, s, out, ko[0], ko[1], ko[2], in, ki[0], ki[1], ki[2], m[0], m[1], m[2],
               ncomp, keep_rest);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void restrict_grid(T* out, const T* in, const Dims& fine, hipStream_t s) {
  int f[3];
  for (int j = 0; j < 3; ++j) {
    f[j] = fine.n[j] > 1 ? 2 : 1;
    if (fine.n[j] % f[j]) throw ArgError("restrict_grid: odd grid size");
  }
  const int64_t Pc = fine.P / (f[0] * f[1] * f[2]);
  prof::launch("k_restrict_grid<" + std::string(prof::tname<T>()) + ">", 1.0 * (fine.P + Pc) * sizeof(T), 0.0,
               k_restrict_grid<T>, grid_for(Pc), dim3(kBlock), 0, s, out, in, fine.n[0], fine.n[1], fine.n[2], f[0],
               f[1], f[2]);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void scaled_diff(T* out, T a, const T* x, const T* y, int64_t n, hipStream_t s) {
  prof::launch(std::string("k_scaled_diff<") + prof::tname<T>() + ">", 3.0 * n * sizeof(T), 0.0, k_scaled_diff<T>, grid_for(n), dim3(kBlock), 0, s, out, a, x, y, n);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void residual_times_grad(T* out, T a, const T* x, const T* y, const T* g1, const Dims& d, hipStream_t s) {
  prof::launch(std::string("k_residual_times_grad<") + prof::tname<T>() + ">", 6.0 * d.P * sizeof(T), 0.0, k_residual_times_grad<T>, grid_for(d.P), dim3(kBlock), 0, s, out, a, x, y, g1, d.P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void coupling_v3(T* out, T a, const T* g1, const T* w, const Dims& d, hipStream_t s) {
  prof::launch(std::string("k_coupling_v3<") + prof::tname<T>() + ">", 9.0 * d.P * sizeof(T), 0.0, k_coupling_v3<T>, grid_for(d.P), dim3(kBlock), 0, s, out, a, g1, w, d.P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void mul(T* out, const T* x, const T* y, int64_t n, hipStream_t s) {
  prof::launch(std::string("k_mul<") + prof::tname<T>() + ">", 3.0 * n * sizeof(T), 0.0, k_mul<T>, grid_for(n), dim3(kBlock), 0, s, out, x, y, n);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void jacobian_det(double* out, const T* Du, int dim, int64_t P, hipStream_t s) {
  (void)dim;
  prof::launch(std::string("k_jacobian<") + prof::tname<T>() + ">", 9.0 * P * sizeof(T) + 8.0 * P, 0.0, k_jacobian<T>, grid_for(P), dim3(kBlock), 0, s, out, Du, P);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void copy_dev(T* dst, const T* src, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  prof::launch(std::string("k_copy<") + prof::tname<T>() + ">", 2.0 * n * sizeof(T), 0.0, k_copy<T>, grid_for(n), dim3(kBlock), 0, s, dst, src, n);
  LDDMM_LAUNCH_CHECK();
}

template <typename T>
void zero(T* p, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  prof::launch(std::string("k_zero<") + prof::tname<T>() + ">", 1.0 * n * sizeof(T), 0.0, k_zero<T>, grid_for(n), dim3(kBlock), 0, s, p, n);
  LDDMM_LAUNCH_CHECK();
}

#define LDDMM_INST(T)                                                                                   \
  template void bl_axpby<T>(T*, T, const T*, T, const T*, int64_t, hipStream_t);                        \
  template void bl_scale_sym<T>(T*, const T*, const double*, int, int64_t, const T*, hipStream_t);      \
  template void bl_div<T>(T*, const T*, const Dims&, hipStream_t);                                      \
  template void characteristics<T>(T*, const T*, const T*, const Dims&, T, int, hipStream_t);           \
  template void interp<T>(T*, const T*, int, const T*, const Dims&, hipStream_t);                       \
  template void prefilter<T>(T*, T*, const T* const*, const T* const*, int, const Dims&, hipStream_t);   \
  template void adjoint_grid_step<T>(T*, const T*, const T*, const T*, const T*, const Dims&, T,        \
                                     hipStream_t);                                                      \
  template void bl_adjoint_step<T>(T*, const T*, const T*, int, const T*, const T*, const Dims&, T,     \
                                   hipStream_t);                                                        \
  template void v3_source<T>(T*, const T*, const T*, const Dims&, hipStream_t);                         \
  template void v1_source<T>(T*, const T*, const T*, const Dims&, hipStream_t);                         \
  template void v1_products<T>(T*, const T*, const T*, const T*, const Dims&, hipStream_t);             \
  template void v3_products<T>(T*, const T*, const T*, const T*, const Dims&, hipStream_t);             \
  template void final_warp<T>(T*, T*, const T*, const T*, const Dims&, hipStream_t);                    \
  template void pull_back<T>(T*, const T*, const T*, const T*, T, int, const Dims&, hipStream_t);        \
  template void node_sum<T>(T*, const T*, const T*, int, int64_t, hipStream_t);                          \
  template void band_copy<T>(T*, const int*, const T*, const int*, const int*, int, bool, hipStream_t);   \
  template void restrict_grid<T>(T*, const T*, const Dims&, hipStream_t);                                 \
  template void rk_adjoint_rhs<T>(T*, const T*, const T*, const T*, const T*, int64_t, hipStream_t);      \
  template void rk_inc_rhs<T>(T*, const T*, const T*, const T*, T, T, const T*, const T*, int64_t,         \
                              hipStream_t);                                                              \
  template void scaled_diff<T>(T*, T, const T*, const T*, int64_t, hipStream_t);                        \
  template void residual_times_grad<T>(T*, T, const T*, const T*, const T*, const Dims&, hipStream_t);  \
  template void coupling_v3<T>(T*, T, const T*, const T*, const Dims&, hipStream_t);                    \
  template void mul<T>(T*, const T*, const T*, int64_t, hipStream_t);                                   \
  template void jacobian_det<T>(double*, const T*, int, int64_t, hipStream_t);                          \
  template void zero<T>(T*, int64_t, hipStream_t);                                                     \
  template void copy_dev<T>(T*, const T*, int64_t, hipStream_t);

LDDMM_INST(float)
LDDMM_INST(double)

}  // namespace lddmm
