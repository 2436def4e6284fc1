// Plane-wise truncated DFT (Section 2.2) on the matrix cores, float.
//
// The 3D transforms are split at the first axis into a band-side stage and a
// plane-side stage, joined by "plane-band" arrays [x0][a1][a2] (one K1 x K2
// block per grid plane x0):
//   iota:  T[x0] = sum_a0 W0[x0][a0] c[a0]            (k_axis0, P part)
//          out[x0][x1][x2] = W1 T[x0] W2^T             (k_expand)
//   pi:    R[x0] = P1 f[x0] P2^T                       (k_reduce)
//          c[a0] = sum_x0 P0[a0][x0] R[x0]             (k_axis0, F part)
// k_axis0 does both first-axis stages in one launch: it finishes a projection
// (with an epilogue out = beta out + alpha r + gamma z) and forms from the
// finished coefficients, or from any band arrays, the plane-band inputs of the
// next expansions, so one semi-Lagrangian step costs expand -> interpolate ->
// reduce -> axis0.
//
// Each wave owns 32 x 32 output tiles of v_mfma_f32_32x32x2f32 (lane l holds
// A[l%32][l/32] and B[l/32][l%32] of a k-step; the accumulator register r of
// lane l holds D[acc_row(r, l)][l%32]).  Every operand load of a k-step is one
// coalesced row segment: the matrices are read in the layout whose rows are the
// contraction index, and grid fields and plane-band arrays are read along their
// contiguous axis.  The two contractions of a plane are chained in registers:
// the accumulator of the first, read as the A operand of the second (lane l%32
// its row, register r its k-step), contracts the first product's row index, so
// no LDS transpose or barrier sits between them.  A contraction's k-steps may
// visit the summation index in any order as long as both operands follow it.
#include "kernels.h"
#include "prof.h"

#include <algorithm>
#include <string>

namespace lddmm {

typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

// row of the 32 x 32 accumulator tile held in register r of a lane
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

__device__ __forceinline__ f32x16 mfma(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void zero16(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = 0.f;
}

// Raw buffer loads: a byte offset per lane (a register that loads at uniform distances share) and an element offset
// uniform across the wave.  The hardware's range check covers the sum of the two and returns 0 at or past the end of
// the buffer, so a tile that runs past the last row of an array reads zeros, as it does with a lane offset of kOut.
// (The tests' short and odd axes give wrong sums where a row past the end reads anything else.)
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr unsigned kOut = 0xFFFFFFF0u;
__device__ __forceinline__ Rsrc rsrc(const float* p, int64_t n) {
  const int64_t bytes = n * 4 < 0x7FFFFFF0 ? n * 4 : 0x7FFFFFF0;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float bload_at(Rsrc r, unsigned voff, unsigned uidx) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)(uidx * 4u), 0));
}

// Values the compiler cannot see are equal across a wave (they derive from the wave index) are moved
// to scalar registers, so pointer tables indexed by them are read with scalar loads.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// ------------------------------------------------------------------ expansion
// One workgroup (4 waves) per (field f, plane x0, x1 block b of 32 rows).  Stage 1,
// V[a2][x1] = sum_a1 T[a1][a2] W1t[a1][x1] (T read along a2, W1t along x1), is split over the waves by
// k-steps and summed in LDS in wave order; stage 2, out[x1][x2] = sum_a2 V[a2][x1] W2t[a2][x2] with V's
// registers as the A operand, takes the x2 tiles wave, wave + 4, ...  Ragged lanes need no test: a
// lane past n1 or n2 reads finite neighbouring entries and its results are not stored, and rows
// a2 >= k2 of V meet rows of W2t past its end, which read as zeros (every plane-band entry a tile can
// reach is written or zero-initialised, so finite).
template <int JB, int KT2>
__global__ __launch_bounds__(256) void k_expand(PlaneExpandArgs a) {
  __shared__ float red[4 * KT2 * 1024];
  constexpr int JW = JB / 4;  // stage-1 k-steps per wave
  const int lane = threadIdx.x & 63, i = lane & 31, kh = lane >> 5;
  const int wave = uniform(threadIdx.x >> 6);
  const int n1 = a.n1, n2 = a.n2, k1 = a.k1, k2 = a.k2;
  const int T2 = (n2 + 31) >> 5;
  const int b = blockIdx.x, x0 = blockIdx.y, f = blockIdx.z;
  const Rsrc rT = rsrc(a.T[f] + x0 * (k1 * k2), (int64_t)(a.n0 - x0) * k1 * k2);
  const Rsrc r1 = rsrc(a.w1t[f], (int64_t)k1 * n1);  // [k1][n1]
  const Rsrc r2 = rsrc(a.w2t[f], (int64_t)k2 * n2);  // [k2][n2]
  float* __restrict__ out = a.out + (size_t)(f * a.n0 + x0) * (size_t)(n1 * n2);
  // stage 1, this wave's k-steps j = wave JW .. wave JW + JW - 1 (a1 = 2 j + kh)
  const int j0 = 2 * JW * wave;
  const unsigned vt = (unsigned)(kh * k2 + i) * 4u, vw = (unsigned)(kh * n1 + b * 32 + i) * 4u;
  float wb[JW], ta[KT2][JW];
#pragma unroll
  for (int u = 0; u < JW; ++u) {
    wb[u] = bload_at(r1, vw, (j0 + 2 * u) * n1);
#pragma unroll
    for (int q = 0; q < KT2; ++q) ta[q][u] = bload_at(rT, vt, (j0 + 2 * u) * k2 + 32 * q);
  }
  // stage-2 operands of the wave's first x2 tile
  float wc[KT2][16];
  auto load_wc = [&](int t) {
    const unsigned v = (unsigned)(4 * kh * n2 + t * 32 + i) * 4u;
#pragma unroll
    for (int q = 0; q < KT2; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) wc[q][r] = bload_at(r2, v, (q * 32 + acc_row(r, 0)) * n2);
  };
  load_wc(wave);
  if (a.y[f]) {
    const Rsrc ry = rsrc(a.y[f] + x0 * (k1 * k2), (int64_t)(a.n0 - x0) * k1 * k2);
    float ty[KT2][JW];
#pragma unroll
    for (int q = 0; q < KT2; ++q)
#pragma unroll
      for (int u = 0; u < JW; ++u) ty[q][u] = bload_at(ry, vt, (j0 + 2 * u) * k2 + 32 * q);
#pragma unroll
    for (int q = 0; q < KT2; ++q)
#pragma unroll
      for (int u = 0; u < JW; ++u) ta[q][u] += a.alpha[f] * ty[q][u];
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x16 V[KT2];
#pragma unroll
  for (int q = 0; q < KT2; ++q) {
    zero16(V[q]);
#pragma unroll
    for (int u = 0; u < JW; ++u) V[q] = mfma(ta[q][u], wb[u], V[q]);
#pragma unroll
    for (int r = 0; r < 16; ++r) red[((wave * KT2 + q) * 16 + r) * 64 + lane] = V[q][r];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < KT2; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int e = (q * 16 + r) * 64 + lane;
      V[q][r] = red[e] + red[KT2 * 1024 + e] + red[2 * KT2 * 1024 + e] + red[3 * KT2 * 1024 + e];
    }
  // stage 2: k-step r of tile q contracts a2 = q 32 + acc_row(r); output rows x1, columns x2
  for (int t2 = wave; t2 < T2; t2 += 4) {
    const int x2 = t2 * 32 + i;
    if (t2 != wave) load_wc(t2);
    f32x16 acc;
    zero16(acc);
#pragma unroll
    for (int q = 0; q < KT2; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc = mfma(V[q][r], wc[q][r], acc);
    if (x2 < n2) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = b * 32 + acc_row(r, lane);
        if (row < n1) out[(unsigned)(row * n2 + x2)] = acc[r];
      }
    }
  }
}

// ------------------------------------------------------------------ reduction
// Grid value of field f at a node of it for the modes: a plain field, or a pointwise product of band-limited fields
// on the product grid.  Loads past the arrays read 0.  A plain field is the caller's and may hold infinities or NaN,
// so the array is field f alone: the next field's values would meet the zeros past P1t's end.
template <int MODE>
struct RedIn {
  Rsrc in, e, divv, G;
  unsigned P, en;
  __device__ __forceinline__ RedIn(const PlaneReduceArgs& a, int f) : P((unsigned)a.P), en((unsigned)a.e_node) {
    if constexpr (MODE == kRedPlain) {
      in = rsrc(a.in + f * a.P, a.P);
    } else {
      const int64_t ne = (MODE == kRedV1Products) ? 1 : (MODE == kRedV1Source || MODE == kRedV3Source) && a.e_node
                         ? (int64_t)(MODE == kRedV1Source ? a.nf : a.nf / 3) * 3 : 3;
      const int ng = MODE == kRedV1Products ? 3 : MODE == kRedV3Products ? 9
                   : MODE == kRedV1Source   ? 3 * a.nf : 3 * a.nf;
      e = rsrc(a.e, (int64_t)ne * a.P);
      G = rsrc(a.G, (int64_t)ng * a.P);
      divv = rsrc(a.divv ? a.divv : a.e, a.P);
    }
  }
  // in two steps, for the node at byte offset v (per lane) plus u elements (uniform): request its values, then combine
  // them
  static constexpr int kRaw = MODE == kRedPlain ? 1 : MODE == kRedV1Products ? 2 : MODE == kRedV3Source ? 7 : 6;
  __device__ __forceinline__ void fetch(int f, unsigned v, unsigned u, float (&x)[kRaw]) const {
    if constexpr (MODE == kRedPlain) {
      x[0] = bload_at(in, v, u);
    } else if constexpr (MODE == kRedV1Products) {  // [e div v, e G0, e G1, e G2]
      x[0] = bload_at(e, v, u);
      x[1] = f == 0 ? bload_at(divv, v, u) : bload_at(G, v, (unsigned)(f - 1) * P + u);
    } else if constexpr (MODE == kRedV3Products) {  // [e_i div v (3), sum_i e_i d_j u_i (3)]
      if (f < 3) {
        x[0] = bload_at(e, v, (unsigned)f * P + u), x[1] = bload_at(divv, v, u);
#pragma unroll
        for (int k = 2; k < 6; ++k) x[k] = 0.f;
      } else {
#pragma unroll
        for (int k = 0; k < 3; ++k)
          x[2 * k] = bload_at(e, v, k * P + u), x[2 * k + 1] = bload_at(G, v, (unsigned)(3 * k + f - 3) * P + u);
      }
    } else {  // node n: -G_n . dv_n, or dv_c - sum_j d_j u_c dv_j (f = 3 n + c)
      const unsigned n = MODE == kRedV1Source ? f : f / 3, c = f - 3 * n;
      const unsigned g = (MODE == kRedV1Source ? 3 * n : 9 * n + 3 * c) * P + u, q = n * en + u;
#pragma unroll
      for (int k = 0; k < 3; ++k) x[2 * k] = bload_at(G, v, g + k * P), x[2 * k + 1] = bload_at(e, v, k * P + q);
      if constexpr (MODE == kRedV3Source) x[6] = bload_at(e, v, c * P + q);
    }
  }
  static __device__ __forceinline__ float combine(const float (&x)[kRaw]) {
    if constexpr (MODE == kRedPlain) return x[0];
    else if constexpr (MODE == kRedV1Products) return x[0] * x[1];
    else if constexpr (MODE == kRedV3Products) return x[0] * x[1] + x[2] * x[3] + x[4] * x[5];
    else if constexpr (MODE == kRedV1Source) return -(x[0] * x[1] + x[2] * x[3] + x[4] * x[5]);
    else return x[6] - (x[0] * x[1] + x[2] * x[3] + x[4] * x[5]);
  }
};

// Finished element e of a plane's band block (field f, plane x0): to the partials, or combined into the output
__device__ __forceinline__ void reduce_store(const PlaneReduceArgs& a, int f, int x0, int e, float r) {
  const int n = a.k1 * a.k2;
  if (a.combine) {  // (at most kMaxFields fields, see plane_reduce; the node sources have more)
    float* out = a.out[f] + (size_t)x0 * n + e;
    *out = a.beta[f] == 0.f ? a.alpha[f] * r : a.beta[f] * *out + a.alpha[f] * r;  // beta 0 never reads out
  } else {
    a.part[(size_t)(f * a.n0 + x0) * n + e] = r;
  }
}

// One workgroup per (field, plane x0); its waves take the tasks (x2 tile t of 32 columns, x1 chunk s of
// 64 rows) of the plane.  Stage A: W[x2][a1] = sum_x1 in[x1][x2] P1t[x1][a1] over the chunk (the field
// read along x2; chunks of JC k-steps alternate between two accumulators, shorter rounding chains);
// stage B: R[a1][a2] += sum_x2 W[x2][a1] P2t[x2][a2], W's registers as the A operand.  Ragged tiles need
// no test: rows x1 >= n1 meet rows of P1t past its end and columns x2 >= n2 rows of P2t past its end,
// which read as zeros, against finite grid entries (or others of the same field, all of whose coefficients they
// reach).  The waves' partial R are summed in LDS in wave order (deterministic) and stored.
template <int MODE, int KT1, int KT2, int WAVES, int CH>
__global__ __launch_bounds__(64 * WAVES) void k_reduce(PlaneReduceArgs a) {
  extern __shared__ float red[];  // [WAVES / 2][KT1 KT2][16][64]
  const int lane = threadIdx.x & 63, i = lane & 31, kh = lane >> 5;
  const int wave = uniform(threadIdx.x >> 6);
  const int f = blockIdx.y, x0 = blockIdx.x;
  const int n1 = a.n1, n2 = a.n2, k1 = a.k1, k2 = a.k2;
  const int T2 = (n2 + 31) >> 5, S1 = (n1 + CH - 1) / CH;
  const RedIn<MODE> src(a, f);
  const Rsrc rp1 = rsrc(a.p1t, (int64_t)n1 * k1), rp2 = rsrc(a.p2t, (int64_t)n2 * k2);
  f32x16 R[KT1][KT2];
#pragma unroll
  for (int p = 0; p < KT1; ++p)
#pragma unroll
    for (int q = 0; q < KT2; ++q) zero16(R[p][q]);
  const unsigned pbase = (unsigned)(x0 * n1 * n2);
  typedef RedIn<MODE> In;
  constexpr int JA = CH / 2;  // stage-A k-steps of a task: rows s CH + 2 j + kh
  // k-steps of a block: the values of 32 loads, half a task of a plain field, requested before the first product
  constexpr int JC = In::kRaw > 2 ? 4 : In::kRaw > 1 ? 8 : JA < 16 ? JA : 16;
  constexpr int NH = JA / JC > 1 ? 2 : 1;  // accumulators (shorter rounding chains)
  unsigned va[KT1], vb[KT2];  // this lane's entry of a row (kh) of P1t, of a row (4 kh) of P2t
#pragma unroll
  for (int p = 0; p < KT1; ++p) va[p] = p * 32 + i < k1 ? (unsigned)(kh * k1 + p * 32 + i) * 4u : kOut;
#pragma unroll
  for (int q = 0; q < KT2; ++q) vb[q] = q * 32 + i < k2 ? (unsigned)(4 * kh * k2 + q * 32 + i) * 4u : kOut;
  for (int task = wave; task < T2 * S1; task += WAVES) {
    const int t = task % T2, s = task / T2;
    const unsigned vx = (unsigned)(kh * n2 + t * 32 + i) * 4u;
    f32x16 W[NH][KT1];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int p = 0; p < KT1; ++p) zero16(W[h][p]);
#pragma unroll
    for (int jc = 0; jc < JA; jc += JC) {
      float xa[JC][In::kRaw], pb[KT1][JC];
#pragma unroll
      for (int j = 0; j < JC; ++j) {
        const int x1 = s * CH + 2 * (jc + j);
        src.fetch(f, vx, pbase + (unsigned)(x1 * n2), xa[j]);
#pragma unroll
        for (int p = 0; p < KT1; ++p) pb[p][j] = bload_at(rp1, va[p], x1 * k1);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int h = (jc / JC) % NH;
#pragma unroll
      for (int j = 0; j < JC; ++j) {
        const float x = In::combine(xa[j]);
#pragma unroll
        for (int p = 0; p < KT1; ++p) W[h][p] = mfma(x, pb[p][j], W[h][p]);
      }
    }
    // stage B: k-step r contracts x2 = t 32 + acc_row(r)
#pragma unroll
    for (int q = 0; q < KT2; ++q) {
      float pc[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) pc[r] = bload_at(rp2, vb[q], (t * 32 + acc_row(r, 0)) * k2);
#pragma unroll
      for (int p = 0; p < KT1; ++p)
#pragma unroll
        for (int r = 0; r < 16; ++r) R[p][q] = mfma(NH == 2 ? W[0][p][r] + W[NH - 1][p][r] : W[0][p][r], pc[r], R[p][q]);
    }
  }
  // the waves' partials summed in a fixed order in NS = WAVES / 2 slots of LDS: waves w < NS store theirs
  // in slot w, waves w >= NS add theirs to slot w - NS, then the slots are summed in order
  constexpr int TILES = KT1 * KT2;
  constexpr int NS = (WAVES + 1) / 2;
  for (int half = 0; half < 2; ++half) {
    if (half == 0 ? wave < NS : wave >= NS) {
      const int slot = half == 0 ? wave : wave - NS;
#pragma unroll
      for (int p = 0; p < KT1; ++p)
#pragma unroll
        for (int q = 0; q < KT2; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float& d = red[((slot * TILES + p * KT2 + q) * 16 + r) * 64 + lane];
            d = half == 0 ? R[p][q][r] : d + R[p][q][r];
          }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < TILES * 16 * 64; e += 64 * WAVES) {
    const int l = e & 63, r = (e >> 6) & 15, tile = e >> 10;
    const int p = tile / KT2, q = tile - p * KT2;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NS; ++w) sum += red[(w * TILES * 16) * 64 + e];
    const int a1 = p * 32 + acc_row(r, l), a2 = q * 32 + (l & 31);
    if (a1 < k1 && a2 < k2) reduce_store(a, f, x0, a1 * k2 + a2, sum);
  }
}

// ------------------------------------------------------------------ bands above 32: half planes
// With a band above 32 on an inner axis the kernels above are bound by the matrix cores.  On an axis of even
// length a basis function of frequency k satisfies w(x + n/2) = (-1)^k w(x), so the coefficients of even and of
// odd frequencies contribute E and O to a node x < n/2 and E + O, E - O to x and x + n/2: half the products, and
// tiles, loads and stores of whole rows as before.  Slots 0, 3, 4, 7, 8, .. of a band hold the even frequencies,
// 1, 2, 5, 6, .. the odd ones (K/2 of each).

// slot of entry j of the even (p = 0) or odd frequencies
__device__ __forceinline__ int half_slot(int j, int p) { return 4 * (j >> 1) + (p ? 1 + (j & 1) : 3 * (j & 1)); }

// Expansion.  One workgroup per (field f, plane x0, block b of 32 rows x1 < n1/2).  Stage 1: wave 2 p + q forms
// V[a2][x1] over the frequencies a1 of parity p for the slots a2 of parity q; the sums and differences over p, by
// LDS, are V at x1 and x1 + n1/2.  Stage 2: a wave per (x2 tile of the half row, half of the rows).
// B1, B2: k-steps over a parity's K/2 slots.  256^3, 64^3 coefficients, three fields: 112 -> 57 us (201 MB at 3.5
// TB/s; with the registers of eight waves a workgroup, two waves a SIMD, 72); 160 x 192 x 160, 40 x 48 x 40: 37 -> 22.
template <int B1, int B2>
__global__ __launch_bounds__(B2 <= 12 ? 512 : 256, B2 <= 12 ? 4 : 3) void k_expand_r2(PlaneExpandArgs a) {
  __shared__ float red[4 * 1024];
  const int lane = threadIdx.x & 63, i = lane & 31, kh = lane >> 5;
  const int wave = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int n1 = a.n1, n2 = a.n2, k1 = a.k1, k2 = a.k2, h1 = n1 >> 1, h2 = n2 >> 1;
  const int T2 = (h2 + 31) >> 5;
  const int b = blockIdx.x, x0 = blockIdx.y, f = blockIdx.z;
  const Rsrc rT = rsrc(a.T[f] + x0 * (k1 * k2), (int64_t)(a.n0 - x0) * k1 * k2);
  const Rsrc r1 = rsrc(a.w1t[f], (int64_t)k1 * n1);  // [k1][n1]
  const Rsrc r2 = rsrc(a.w2t[f], (int64_t)k2 * n2);  // [k2][n2]
  float* __restrict__ out = a.out + (size_t)(f * a.n0 + x0) * (size_t)(n1 * n2);
  float wc[2][B2];
  auto load_wc = [&](int t) {
    const unsigned v = (unsigned)(half_slot(acc_row(0, lane), 0) * n2 + t * 32 + i) * 4u;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < B2; ++r) wc[q][r] = bload_at(r2, v, half_slot(acc_row(r, 0), q) * n2);
  };
  if (wave < 4) {
    const int p = wave >> 1, q = wave & 1, row = half_slot(kh, p);
    const unsigned vt = (unsigned)(row * k2 + half_slot(i, q)) * 4u, vw = (unsigned)(row * n1 + b * 32 + i) * 4u;
    float ta[B1], wb[B1];
#pragma unroll
    for (int j = 0; j < B1; ++j) {
      ta[j] = bload_at(rT, vt, 4 * j * k2);
      wb[j] = bload_at(r1, vw, 4 * j * n1);
    }
    if (a.y[f]) {
      const Rsrc ry = rsrc(a.y[f] + x0 * (k1 * k2), (int64_t)(a.n0 - x0) * k1 * k2);
      float ty[B1];
#pragma unroll
      for (int j = 0; j < B1; ++j) ty[j] = bload_at(ry, vt, 4 * j * k2);
#pragma unroll
      for (int j = 0; j < B1; ++j) ta[j] += a.alpha[f] * ty[j];
    }
    load_wc(wave >> 1);
    f32x16 V;
    zero16(V);
#pragma unroll
    for (int j = 0; j < B1; ++j) V = mfma(ta[j], wb[j], V);
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = V[r];
  } else {
    load_wc(wave >> 1);
  }
  __syncthreads();
  for (int task = wave; task < 2 * T2; task += nw) {
    const int t = task >> 1, sd = task & 1, x2 = t * 32 + i;
    if (task != wave) load_wc(t);
    f32x16 E, O;
    zero16(E);
    zero16(O);
#pragma unroll
    for (int r = 0; r < B2; ++r) {
      const float e0 = red[r * 64 + lane], e1 = red[(16 + r) * 64 + lane];
      const float o0 = red[(32 + r) * 64 + lane], o1 = red[(48 + r) * 64 + lane];
      E = mfma(sd ? e0 - o0 : e0 + o0, wc[0][r], E);
      O = mfma(sd ? e1 - o1 : e1 + o1, wc[1][r], O);
    }
    if (x2 < h2) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = b * 32 + acc_row(r, lane);
        if (row < h1) {
          const unsigned o = (unsigned)((row + sd * h1) * n2 + x2);
          out[o] = E[r] + O[r];
          out[o + h2] = E[r] - O[r];
        }
      }
    }
  }
}

// ------------------------------------------------------------------ bands above 32: half planes, reduction
// The transpose of k_expand_r2: sums and differences of the rows x1, x1 + n1/2 and of the columns x2, x2 + n2/2
// feed the even and odd frequencies.  One workgroup per (field, plane x0); a wave takes the frequencies a1 of one
// parity and the tasks (x2 tile t of the half row, chunk of the half column) wave / 2, wave / 2 + nw / 2, ..:
// stage A, W[x2][a1] for either parity of a2; stage B, R[a1][a2] += sum_x2 W[x2][a1] P2t[x2][a2].  Its registers
// leave room for four waves a SIMD, which hide each other's loads (both parities in one wave, its loads a block
// ahead: two waves, slower for plain fields).  256^3, 64^3 coefficients, three fields: 147 -> 70 us (201 MB at 2.9
// TB/s), 160 x 192 x 160, 40 x 48 x 40: 49 -> 29, its products 31 -> 18.
template <int MODE>
__global__ __launch_bounds__(512, 4) void k_reduce_r2(PlaneReduceArgs a, int chunk) {
  extern __shared__ float red[];  // [waves][2][16][64]
  typedef RedIn<MODE> In;
  constexpr int JC = MODE == kRedPlain ? 8 : In::kRaw == 2 ? 4 : 1;  // k-steps of a block
  const int lane = threadIdx.x & 63, i = lane & 31, kh = lane >> 5;
  const int wave = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6, p = wave & 1;
  const int f = blockIdx.y, x0 = blockIdx.x;
  const int n1 = a.n1, n2 = a.n2, k1 = a.k1, k2 = a.k2, h1 = n1 >> 1, h2 = n2 >> 1;
  const int T2 = (h2 + 31) >> 5, S1 = (h1 + chunk - 1) / chunk;
  const In src(a, f);
  const Rsrc rp1 = rsrc(a.p1t, (int64_t)n1 * k1), rp2 = rsrc(a.p2t, (int64_t)n2 * k2);
  const unsigned up = (unsigned)(h1 * n2), plane = (unsigned)(x0 * n1 * n2);
  const float sg = p ? -1.f : 1.f;
  const int sl = half_slot(i, p);
  const unsigned va = sl < k1 ? (unsigned)(kh * k1 + sl) * 4u : kOut;  // this lane's entry of a row (kh) of P1t
  f32x16 R[2];
  zero16(R[0]);
  zero16(R[1]);
  for (int task = wave >> 1; task < T2 * S1; task += nw >> 1) {
    const int t = task % T2, c0 = (task / T2) * chunk, c1 = min(h1, c0 + chunk);
    const unsigned vx = t * 32 + i < h2 ? (unsigned)(kh * n2 + t * 32 + i) * 4u : kOut;
    f32x16 W[2];
    zero16(W[0]);
    zero16(W[1]);
    // k-step j of a block: rows j0 + 2 j + kh
    for (int j0 = c0; j0 < c1; j0 += 2 * JC) {
      float v[JC][4][In::kRaw], pb[JC];
#pragma unroll
      for (int j = 0; j < JC; ++j) {
        const bool row = j0 + 2 * j + kh < c1;
        const unsigned o = row ? vx : kOut, u = plane + (unsigned)((j0 + 2 * j) * n2);
        src.fetch(f, o, u, v[j][0]);
        src.fetch(f, o, u + h2, v[j][1]);
        src.fetch(f, o, u + up, v[j][2]);
        src.fetch(f, o, u + up + h2, v[j][3]);
        pb[j] = bload_at(rp1, row ? va : kOut, (unsigned)((j0 + 2 * j) * k1));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < JC; ++j) {
        const float u0 = fmaf(sg, In::combine(v[j][2]), In::combine(v[j][0]));
        const float u1 = fmaf(sg, In::combine(v[j][3]), In::combine(v[j][1]));
        W[0] = mfma(u0 + u1, pb[j], W[0]);
        W[1] = mfma(u0 - u1, pb[j], W[1]);
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int sl2 = half_slot(i, q);
      const unsigned vb = sl2 < k2 ? (unsigned)(4 * kh * k2 + sl2) * 4u : kOut;
      float pc[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = t * 32 + acc_row(r, 0);
        pc[r] = bload_at(rp2, row + 4 * kh < h2 ? vb : kOut, (unsigned)(row * k2));
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) R[q] = mfma(W[q][r], pc[r], R[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[((wave * 2 + q) * 16 + r) * 64 + lane] = R[q][r];
  __syncthreads();
  // the sum over the waves of a parity, in order
  for (int e = threadIdx.x; e < 4096; e += blockDim.x) {
    const int l = e & 63, r = (e >> 6) & 15, pp = e >> 11;
    float sum = red[e];
    for (int w = 2; w < nw; w += 2) sum += red[(w + pp) * 2048 + (e & 2047)];
    const int s1 = half_slot(acc_row(r, l), pp), s2 = half_slot(l & 31, (e >> 10) & 1);
    if (s1 < k1 && s2 < k2) reduce_store(a, f, x0, s1 * k2 + s2, sum);
  }
}

// ------------------------------------------------------------------ product-grid step
// Expansion and product reduction of one plane in one pass, for the products of a band-limited
// field e~ (1 or 3 components, plane-band inputs T) with node fields on the product grid:
//   part[f][x0] = P1 (prod_f(x0, ., .)) P2^T,  prod_f = e div v, e G_j  (MODE kRedV1Products)
//                                              e_c div v, sum_i e_i G_{3i+j}  (kRedV3Products).
// One workgroup per (output field f, plane x0); wave w owns the grid tile (x1 tile s, x2 tile t) of
// 32 x 32 nodes.  It expands the e components f needs on its tile (V = T W1t, then D = V^T W2t, the
// accumulator of the first read as the A operand of the second), multiplies by the node fields in
// registers, and contracts the tile with P1 over its rows (the product's registers as the A operand)
// and with P2 over its columns; the tiles' partials are summed in LDS in wave order.  The expanded
// field never goes to memory.  Ragged tiles need no test, as in the separate kernels: grid entries past
// n1 / n2 are finite and meet rows of P1t / P2t past their ends, which read as zeros.
template <int MODE>
__global__ __launch_bounds__(512) void k_prod_plane(ProdPlaneArgs a) {
  extern __shared__ float red[];  // [ceil(waves / 2)][16][64]
  constexpr int NE = MODE == kRedV1Products ? 1 : 3;
  const int lane = threadIdx.x & 63, i = lane & 31, kh = lane >> 5;
  const int wave = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int n1 = a.n1, n2 = a.n2, k1 = a.k1, k2 = a.k2;
  const int T2 = (n2 + 31) >> 5;
  const int f = blockIdx.x / a.n0, x0 = blockIdx.x - f * a.n0;
  const int s = wave / T2, t = wave - s * T2;
  const unsigned P = (unsigned)a.P;
  const Rsrc r1 = rsrc(a.w1t, (int64_t)k1 * n1), r2 = rsrc(a.w2t, (int64_t)k2 * n2);
  const Rsrc rp1 = rsrc(a.p1t, (int64_t)n1 * k1), rp2 = rsrc(a.p2t, (int64_t)n2 * k2);
  const Rsrc rdiv = rsrc(a.divv, a.P), rG = rsrc(a.G, (int64_t)(MODE == kRedV1Products ? 3 : 9) * a.P);
  // the e components this output reads: V1 e; V3 f < 3 e_f, f >= 3 all three
  const int c0 = (MODE == kRedV3Products && f < 3) ? f : 0;
  const int ne = (MODE == kRedV3Products && f >= 3) ? 3 : 1;
  // every operand is requested before the first product, in the order of use
  float ta[NE][16], w1[16], w2[16], gf[NE][16], p1[16], p2[16];
  const unsigned vt = (unsigned)(kh * k2 + i) * 4u, v1 = (unsigned)(kh * n1 + s * 32 + i) * 4u;
  const unsigned vg = (unsigned)(4 * kh * n2 + t * 32 + i) * 4u;  // (a row of W2t too)
  const unsigned vp1 = i < k1 ? (unsigned)(4 * kh * k1 + i) * 4u : kOut, vp2 = i < k2 ? (unsigned)(4 * kh * k2 + i) * 4u : kOut;
#pragma unroll
  for (int c = 0; c < NE; ++c) {
    const int cc = c < ne ? c0 + c : c0;
    const Rsrc rT = rsrc(a.T[cc] + x0 * (k1 * k2), (int64_t)(a.n0 - x0) * k1 * k2);
#pragma unroll
    for (int j = 0; j < 16; ++j) ta[c][j] = c < ne ? bload_at(rT, vt, 2 * j * k2) : 0.f;
    if (c == 0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) w1[j] = bload_at(r1, v1, 2 * j * n1);
#pragma unroll
      for (int r = 0; r < 16; ++r) w2[r] = bload_at(r2, vg, acc_row(r, 0) * n2);
    }
    // the node field that multiplies e component c: div v, G_{f-1} (V1) or div v, G_{3 c + f - 3} (V3)
    const bool dv = MODE == kRedV1Products ? f == 0 : f < 3;
    const unsigned g = (unsigned)(x0 * n1 * n2) + (dv ? 0u : (unsigned)(MODE == kRedV1Products ? f - 1 : 3 * c + f - 3) * P);
    const Rsrc rg = dv ? rdiv : rG;
#pragma unroll
    for (int r = 0; r < 16; ++r) gf[c][r] = c < ne ? bload_at(rg, vg, g + (unsigned)((s * 32 + acc_row(r, 0)) * n2)) : 0.f;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) p1[r] = bload_at(rp1, vp1, (s * 32 + acc_row(r, 0)) * k1);
#pragma unroll
  for (int r = 0; r < 16; ++r) p2[r] = bload_at(rp2, vp2, (t * 32 + acc_row(r, 0)) * k2);
  __builtin_amdgcn_sched_barrier(0);
  f32x16 Y;
  zero16(Y);
#pragma unroll
  for (int c = 0; c < NE; ++c) {
    if (c >= ne) break;
    f32x16 V, D;
    zero16(V);
    zero16(D);
    // V[a2][x1] = sum_a1 T[a1][a2] W1t[a1][x1], D[x1][x2] = sum_a2 V[a2][x1] W2t[a2][x2]
#pragma unroll
    for (int j = 0; j < 16; ++j) V = mfma(ta[c][j], w1[j], V);
#pragma unroll
    for (int r = 0; r < 16; ++r) D = mfma(V[r], w2[r], D);
#pragma unroll
    for (int r = 0; r < 16; ++r) Y[r] += D[r] * gf[c][r];
  }
  // W[x2][a1] = sum_x1 Y[x1][x2] P1t[x1][a1] over the tile's rows, R[a1][a2] = sum_x2 W[x2][a1] P2t[x2][a2] over
  // its columns
  f32x16 W, R;
  zero16(W);
  zero16(R);
#pragma unroll
  for (int r = 0; r < 16; ++r) W = mfma(Y[r], p1[r], W);
#pragma unroll
  for (int r = 0; r < 16; ++r) R = mfma(W[r], p2[r], R);
  // partials summed in LDS in a fixed order: waves w < ns store theirs in slot w, then waves w >= ns add
  // theirs to slot w - ns, then the slots are summed in order (ns = ceil(nw / 2) slots of LDS)
  const int ns = (nw + 1) >> 1;
  for (int half = 0; half < 2; ++half) {
    if (half == 0 ? wave < ns : wave >= ns) {
      float* d = red + (half == 0 ? wave : wave - ns) * 1024 + lane;
#pragma unroll
      for (int r = 0; r < 16; ++r) d[r * 64] = half == 0 ? R[r] : d[r * 64] + R[r];
    }
    __syncthreads();
  }
  float* __restrict__ part = a.part + (size_t)blockIdx.x * (k1 * k2);
  for (int e = threadIdx.x; e < 1024; e += blockDim.x) {
    const int l = e & 63, a1 = acc_row(e >> 6, l), a2 = l & 31;
    float sum = 0.f;
    for (int w = 0; w < ns; ++w) sum += red[w * 1024 + e];
    if (a1 < k1 && a2 < k2) part[a1 * k2 + a2] = sum;
  }
}

// ------------------------------------------------------------------ first axis
// Workgroup (column tile of 32 band columns (a1, a2), row y) with the descriptor row[y] resolved on the host: F of
// field y (y < nin): r[a0][c] = sum_x0 P0t[x0][a0] part[x0][c] (x0 in chunks of 8 dealt to the 8 waves, summed in
// LDS in wave order), out = beta in + alpha r + gamma z + ysym y; then up to two P outputs
// T[x0'][c] = sum_a0 W0t[a0][x0'] (c1 g1 + c2 g2 + cf fin)[a0][c], fin the field just finished, a wave per output
// and tile of 32 rows x0'.  A launch is a few dozen workgroups and waits for memory twice, so what bounds it is
// latency and the fetch of its code: every operand that does not depend on F is requested at the start, each
// element of a band array by one thread (the sources of P meet in LDS), loads and stores of a lane share one offset
// register, and rows past the end of an operand read as zeros.  128^3 with 32^3 coefficients: 7.6 -> 5.2 us
// with one field, 8.3 -> 5.8 with four (from 14 KB of code at 32-bit offsets per load and four waves).
template <int KT0, int JB>
__global__ __launch_bounds__(512) void k_axis0(Axis0Kernel a) {
  __shared__ float red[8 * KT0 * 1024];
  __shared__ float src[2][KT0 * 1024];  // the sources of the P outputs, [a0][32 columns]
  constexpr int CB = 3, M = 2 * KT0;    // chunks of a batch; band elements of a thread
  const int lane = threadIdx.x & 63, i = lane & 31, kh = lane >> 5;
  const int wave = uniform(threadIdx.x >> 6);
  const int C = a.C, k0 = a.k0, c = blockIdx.x * 32 + i;
  const Axis0Kernel::Row& row = a.row[blockIdx.y];
  const bool hasF = (int)blockIdx.y < a.nin;
  const Axis0Kernel::Field& F = a.fld[hasF ? blockIdx.y : 0];
  const int np = row.np, Q = k0 * C;
  // this thread's band elements: rows elem(m) + 4 kh of column c
  const unsigned ve = c < C ? (unsigned)(4 * kh * C + c) * 4u : kOut;
  auto elem = [&](int m) { return 32 * (m >> 1) + acc_row(wave + 8 * (m & 1), 0); };
  auto request = [&](float (&x)[M], const float* p) {  // p may be null: zeros
#pragma unroll
    for (int m = 0; m < M; ++m) x[m] = 0.f;
    if (p) {
      const Rsrc r = rsrc(p, Q);
#pragma unroll
      for (int m = 0; m < M; ++m) x[m] = bload_at(r, ve, elem(m) * C);
    }
  };
  float g[2][2][M], in[M], z[M], y[M];
  double sym[M];
#pragma unroll
  for (int u = 0; u < 2; ++u) request(g[u][0], row.p[u].g1), request(g[u][1], row.p[u].g2);
  if (hasF) {
    request(in, F.beta != 0.f ? F.in : nullptr);  // (an output buffer need not hold finite values before)
    request(z, F.z);
    request(y, F.y);
    if (F.y)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int a0 = elem(m) + 4 * kh;
        sym[m] = F.ysym[a0 < k0 && c < C ? a0 * C + c : 0];
      }
  }
  // the first task's rows of W0t
  auto tiles = [&](int u) { return (row.p[u].n0t + 31) >> 5; };
  const int t0 = tiles(0), ntask = np ? t0 + (np > 1 ? tiles(1) : 0) : 0;
  float w[JB];
  auto load_w = [&](int task) {
    const Axis0Kernel::Out& o = row.p[task >= t0];
    const Rsrc r = rsrc(o.w0t, (int64_t)k0 * o.n0t);
    const unsigned v = (unsigned)(kh * o.n0t + (task - (task >= t0 ? t0 : 0)) * 32 + i) * 4u;
#pragma unroll
    for (int j = 0; j < JB; ++j) w[j] = bload_at(r, v, 2 * j * o.n0t);
  };
  if (wave < ntask) load_w(wave);
  float fin[M] = {};
  if (hasF) {
    const int nch = (a.n0 + 7) >> 3;
    const Rsrc rpart = rsrc(F.part, (int64_t)a.n0 * C), rp0 = rsrc(a.p0t, (int64_t)a.n0 * k0);
    const unsigned vp = (unsigned)(4 * kh * C + c) * 4u, va = (unsigned)(4 * kh * k0 + i) * 4u;
    f32x16 acc[KT0];
#pragma unroll
    for (int p = 0; p < KT0; ++p) zero16(acc[p]);
    // k-step j of a chunk: rows 8 ch + j + 4 kh; a wave's CB chunks are requested at once
    for (int ch = wave; ch < nch; ch += 8 * CB) {
      float bv[CB][4], av[CB][KT0][4];
#pragma unroll
      for (int u = 0; u < CB; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int x0 = (ch + 8 * u) * 8 + j;
          bv[u][j] = bload_at(rpart, x0 + 4 * kh < a.n0 ? vp : kOut, x0 * C);
#pragma unroll
          for (int p = 0; p < KT0; ++p) av[u][p][j] = bload_at(rp0, x0 + 4 * kh < a.n0 ? va + 128u * p : kOut, x0 * k0);
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < CB; ++u)
        if (ch + 8 * u < nch) {
#pragma unroll
          for (int p = 0; p < KT0; ++p)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[p] = mfma(av[u][p][j], bv[u][j], acc[p]);
        }
    }
#pragma unroll
    for (int p = 0; p < KT0; ++p)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[((wave * KT0 + p) * 16 + r) * 64 + lane] = acc[p][r];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int e = threadIdx.x + 512 * m, a0 = elem(m) + 4 * kh;
      float sum = red[e];
#pragma unroll
      for (int q = 1; q < 8; ++q) sum += red[q * KT0 * 1024 + e];
      const bool ok = a0 < k0 && c < C;
      float v = F.beta * in[m] + F.gamma * z[m];
      if (F.y) v += static_cast<float>(sym[m]) * y[m];
      v = ok ? F.alpha * sum + v : 0.f;
      if (ok) {
        F.out[a0 * C + c] = v;
        if (F.out2) F.out2[a0 * C + c] = F.s2 * v;
      }
      fin[m] = v;
    }
  }
  if (np == 0) return;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const Axis0Kernel::Out& o = row.p[u];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      float v = o.c1 * g[u][0][m] + o.c2 * g[u][1][m];
      if (o.cf != 0.f) v += o.cf * fin[m];
      src[u][(elem(m) + 4 * kh) * 32 + i] = v;
    }
  }
  __syncthreads();
  for (int task = wave; task < ntask; task += 8) {
    if (task != wave) load_w(task);
    const int u = task >= t0, rt = task - (u ? t0 : 0);
    const Axis0Kernel::Out& o = row.p[u];
    f32x16 acc;
    zero16(acc);
#pragma unroll
    for (int j = 0; j < JB; ++j) acc = mfma(w[j], src[u][(2 * j + kh) * 32 + i], acc);
    const Rsrc rT = rsrc(o.T, (int64_t)o.n0t * C);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int x0 = rt * 32 + acc_row(r, 0);
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)acc[r]), rT,
                                            (int)(x0 + 4 * kh < o.n0t ? ve : kOut), x0 * C * 4, 0);
    }
  }
}

}  // namespace

bool planes_ok(const Dims& d) {
  // 32-bit offsets within a field and within a first-axis stage
  return d.k[0] <= 64 && d.k[1] <= 64 && d.k[2] <= 64 && (d.k[0] == 1 || d.k[0] % 2 == 0) && d.k[1] % 2 == 0 &&
         d.k[2] % 2 == 0 && d.P < (int64_t(1) << 31) && (int64_t)d.n[0] * d.k[1] * d.k[2] < (int64_t(1) << 31);
}

// half planes on even inner axes where a band reaches beyond `above`: the expansion from 18 slots on (128^3, 32^3,
// two fields 9.8 -> 7.6 us, six 21.8 -> 16.3), the reduction above 32 (its tile's columns are a parity's slots, half
// of them empty at 32: 6.8 -> 11.1)
static bool half_planes(int n1, int n2, int k1, int k2, int above) {
  return (k1 > above || k2 > above) && k1 <= 64 && k2 <= 64 && k1 % 2 == 0 && k2 % 2 == 0 && n1 % 2 == 0 && n2 % 2 == 0;
}

void plane_expand(const PlaneExpandArgs& a, hipStream_t s) {
  const int B1 = ceil_div(a.n1, 32);
  if (a.n0 > 65535 || a.nf > 65535) throw ArgError("plane_expand: grid too large");
  const double bytes = 4.0 * a.nf * ((double)a.n0 * a.k1 * a.k2 + (double)a.n0 * a.n1 * a.n2);
  const double flops = 2.0 * a.nf * a.n0 * ((double)a.k1 * a.k2 * a.n1 + (double)a.n1 * a.k2 * a.n2);
  dim3 g(B1, a.n0, a.nf);
  if (half_planes(a.n1, a.n2, a.k1, a.k2, 16)) {
    const dim3 gh(ceil_div(a.n1 / 2, 32), a.n0, a.nf);
    const int waves = std::min(a.k2 <= 48 ? 8 : 4, std::max(4, 2 * ceil_div(a.n2 / 2, 32)));
    auto half = [&](auto kern) { prof::launch("k_expand", bytes, flops, kern, gh, dim3(64 * waves), 0, s, a); };
    if (a.k1 <= 32 && a.k2 <= 32) half(k_expand_r2<8, 8>);
    else if (a.k1 <= 48 && a.k2 <= 48) half(k_expand_r2<12, 12>);
    else if (a.k1 <= 48) half(k_expand_r2<12, 16>);
    else if (a.k2 <= 48) half(k_expand_r2<16, 12>);
    else half(k_expand_r2<16, 16>);
    LDDMM_LAUNCH_CHECK();
    return;
  }
  auto go = [&](auto kern) { prof::launch("k_expand", bytes, flops, kern, g, dim3(256), 0, s, a); };
  if (a.k2 <= 32) {
    if (a.k1 <= 16) go(k_expand<8, 1>); else if (a.k1 <= 32) go(k_expand<16, 1>); else go(k_expand<32, 1>);
  } else {
    if (a.k1 <= 16) go(k_expand<8, 2>); else if (a.k1 <= 32) go(k_expand<16, 2>); else go(k_expand<32, 2>);
  }
  LDDMM_LAUNCH_CHECK();
}

template <int MODE>
static void reduce_mode(const PlaneReduceArgs& a, hipStream_t s, double bytes, double flops) {
  const int kt1 = a.k1 > 32 ? 2 : 1, kt2 = a.k2 > 32 ? 2 : 1;
  const dim3 g(a.n0, a.nf);
  const char* nm = MODE == kRedPlain ? "k_reduce" : "k_reduce_products";
  // tasks of 64 rows (16-wave workgroups with 32-row tasks measured slower); 8 waves (4 for two band tiles
  // per axis: 8 slowed the product modes of the 40x48x40 band from 29 to 54 us), their partials in half as
  // many slots of LDS (KT1 KT2 x 4 KB each)
  // Small planes (the 48 x 48 product grid of a 32-wide band: two 64-row tasks for eight waves) take
  // 16-row tasks instead, one per wave: each wave's chain of dependent load groups is then one group
  // long instead of four.
  if (half_planes(a.n1, a.n2, a.k1, a.k2, 32)) {  // (a parity of a 32-slot band would fill half a tile)
    // two waves (the parities of a1) per x2 tile of the half row and chunk of the half column, up to eight;
    // chunks of at least 16 rows
    const int th = ceil_div(a.n2 / 2, 32), h1 = a.n1 / 2;
    const int parts = std::max(1, std::min(4 / th, h1 / 16));
    const int waves = std::min(8, 2 * th * parts);
    prof::launch(nm, bytes, flops, k_reduce_r2<MODE>, g, dim3(64 * waves), waves * 2 * 1024 * 4, s, a,
                 ceil_div(h1, parts));
    LDDMM_LAUNCH_CHECK();
    return;
  }
  const int t2 = ceil_div(a.n2, 32);
  const bool small = 2 * t2 * ceil_div(a.n1, 64) <= 8 && t2 * ceil_div(a.n1, 16) <= 8;
  if (kt1 == 1 && kt2 == 1 && small)
    prof::launch(nm, bytes, flops, k_reduce<MODE, 1, 1, 8, 16>, g, dim3(512), 4 * 1024 * 4, s, a);
  else if (kt1 == 1 && kt2 == 1)
    prof::launch(nm, bytes, flops, k_reduce<MODE, 1, 1, 8, 64>, g, dim3(512), 4 * 1024 * 4, s, a);
  else if (kt1 == 1)
    prof::launch(nm, bytes, flops, k_reduce<MODE, 1, 2, 8, 64>, g, dim3(512), 4 * 2048 * 4, s, a);
  else if (kt2 == 1)
    prof::launch(nm, bytes, flops, k_reduce<MODE, 2, 1, 8, 64>, g, dim3(512), 4 * 2048 * 4, s, a);
  else
    prof::launch(nm, bytes, flops, k_reduce<MODE, 2, 2, 4, 64>, g, dim3(256), 2 * 4096 * 4, s, a);
  LDDMM_LAUNCH_CHECK();
}

void plane_reduce(const PlaneReduceArgs& a, hipStream_t s) {
  const double flops = 2.0 * a.nf * a.n0 * ((double)a.n1 * a.n2 * a.k1 + (double)a.k1 * a.n2 * a.k2);
  const double bytes = 4.0 * a.nf * a.n0 * ((double)a.n1 * a.n2 + (double)a.k1 * a.k2);
  if (a.P >= (int64_t(1) << 31)) throw ArgError("plane_reduce: field too large");
  if (a.combine && a.nf > kMaxFields) throw ArgError("plane_reduce: too many fields to combine");
  switch (a.mode) {
    case kRedPlain: return reduce_mode<kRedPlain>(a, s, bytes, flops);
    case kRedV1Products: return reduce_mode<kRedV1Products>(a, s, bytes, flops);
    case kRedV3Products: return reduce_mode<kRedV3Products>(a, s, bytes, flops);
    case kRedV1Source: return reduce_mode<kRedV1Source>(a, s, bytes, flops);
    case kRedV3Source: return reduce_mode<kRedV3Source>(a, s, bytes, flops);
    default: throw ArgError("plane_reduce: unknown mode");
  }
}

// one wave per 32 x 32 tile of a plane (at most 8), their partials in ceil(tiles / 2) slots of 4 KB of
// LDS.  The fused pass is chosen for inner bands of at most 32 (one band tile per axis): with two,
// every workgroup's repeated expansions (each output field's workgroup expands the e components it
// reads) cost more than the separate kernels save (160x192x160 / 40x48x40 deformation state: 46 us
// per fused launch against 30 us for the separate reduction).
static bool prod_plane_fits(int n1, int n2, int k1, int k2) {
  return ceil_div(n1, 32) * ceil_div(n2, 32) <= 8 && k1 <= 32 && k2 <= 32;
}
bool prod_plane_ok(const Dims& d) { return planes_ok(d) && prod_plane_fits(d.n[1], d.n[2], d.k[1], d.k[2]); }

void plane_prod(const ProdPlaneArgs& a, hipStream_t s) {
  if (!prod_plane_fits(a.n1, a.n2, a.k1, a.k2)) throw ArgError("plane_prod: plane or band too large");
  const int tiles = ceil_div(a.n1, 32) * ceil_div(a.n2, 32);
  if (a.P >= (int64_t(1) << 31)) throw ArgError("plane_prod: field too large");
  const int nf = a.mode == kRedV1Products ? 4 : 6;
  const int ne = a.mode == kRedV1Products ? 1 : 3;
  const double bytes = 4.0 * a.n0 * (ne * (double)a.k1 * a.k2 + nf * (double)a.k1 * a.k2) +
                       4.0 * a.P * (a.mode == kRedV1Products ? 4 : 10);
  const double flops = 2.0 * nf * a.n0 *
                       ((double)a.k1 * a.k2 * a.n1 + (double)a.n1 * a.k2 * a.n2 + (double)a.n1 * a.n2 * a.k1 +
                        (double)a.k1 * a.n2 * a.k2);
  dim3 g(static_cast<unsigned>(nf * a.n0));
  const dim3 b(64 * tiles);
  const size_t lds = (size_t)((tiles + 1) / 2) * 4096;
  auto go = [&](auto kern) { prof::launch("k_prod_plane", bytes, flops, kern, g, b, lds, s, a); };
  if (a.mode == kRedV1Products) go(k_prod_plane<kRedV1Products>);
  else if (a.mode == kRedV3Products) go(k_prod_plane<kRedV3Products>);
  else throw ArgError("plane_prod: unknown mode");
  LDDMM_LAUNCH_CHECK();
}

void plane_axis0(const Axis0Args& a, hipStream_t s) {
  if (a.nin > kMaxFields || a.nout > kMaxFields) throw ArgError("plane_axis0: too many fields");
  if (a.k0 > 64) throw ArgError("plane_axis0: band above 64");
  // descriptor rows: one per finished field (with the P outputs that read it), then one per P output
  // that reads band arrays only
  Axis0Kernel k{};
  k.p0t = a.p0t, k.n0 = a.n0, k.k0 = a.k0, k.C = a.C, k.nin = a.nin;
  for (int f = 0; f < a.nin; ++f) {
    Axis0Kernel::Field& F = k.fld[f];
    F.part = a.part[f], F.out = a.out[f], F.in = a.in[f] ? a.in[f] : a.out[f], F.out2 = a.out2[f];
    F.z = a.z[f];
    F.y = a.y[f], F.ysym = a.y[f] ? a.ysym[f] : nullptr;
    if (F.y && !F.ysym) throw ArgError("plane_axis0: a symbol-weighted term needs its symbol");
    F.alpha = a.alpha[f], F.beta = a.beta[f], F.gamma = a.z[f] ? a.gamma[f] : 0.f;
    F.s2 = a.s2[f] != 0.f ? a.s2[f] : 1.f;
  }
  int nrow = a.nin;
  double bytes = 4.0 * a.nin * ((double)a.n0 + a.k0) * a.C, flops = 2.0 * a.nin * a.k0 * a.n0 * (double)a.C;
  for (int g = 0; g < a.nout; ++g) {
    const Axis0Out& o = a.o[g];
    const int src = std::max(o.s1, o.s2);
    if (src >= a.nin) throw ArgError("plane_axis0: a P source names an unfinished field");
    if (o.s1 >= 0 && o.s2 >= 0 && o.s1 != o.s2) throw ArgError("plane_axis0: one finished field per P output");
    Axis0Kernel::Row* r;
    if (src >= 0) {
      r = &k.row[src];
      if (r->np >= 2) throw ArgError("plane_axis0: at most two P outputs per finished field");
    } else {
      if (nrow >= Axis0Kernel::kRows) throw ArgError("plane_axis0: too many P outputs");
      r = &k.row[nrow++];
    }
    Axis0Kernel::Out& p = r->p[r->np++];
    p.w0t = o.w0t, p.T = o.T, p.n0t = o.n0t;
    p.g1 = o.g1, p.c1 = o.g1 ? o.c1 : 0.f;
    p.g2 = o.g2, p.c2 = o.g2 ? o.c2 : 0.f;
    p.cf = (o.s1 >= 0 ? o.c1 : 0.f) + (o.s2 >= 0 ? o.c2 : 0.f);
    bytes += 4.0 * (double)o.n0t * a.C;
    flops += 2.0 * o.n0t * a.k0 * (double)a.C;
  }
  if (nrow == 0) return;
  dim3 g(ceil_div(a.C, 32), nrow);
  const std::string nm = "k_axis0[" + std::to_string(a.nin) + "F" + std::to_string(a.nout) + "P]";
  auto go = [&](auto kern) { prof::launch(nm, bytes, flops, kern, g, dim3(512), 0, s, k); };
  if (a.k0 <= 16) go(k_axis0<1, 8>);
  else if (a.k0 <= 32) go(k_axis0<1, 16>);
  else if (a.k0 <= 48) go(k_axis0<2, 24>);
  else go(k_axis0<2, 32>);
  LDDMM_LAUNCH_CHECK();
}

}  // namespace lddmm
