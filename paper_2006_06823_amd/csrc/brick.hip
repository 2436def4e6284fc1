// Tricubic B-spline interpolation at SL departure points through LDS bricks
// (float, 3D grids).
//
// A workgroup owns a tile of output nodes and stages, per coefficient field, the tile plus two nodes on
// every side into LDS (16-byte loads, periodically wrapped).  A thread owns four neighbours of a row.  At
// the SL step sizes of the configurations (about 0.8 voxel) a departure point lies less than a voxel from
// its node, so its 4 x 4 x 4 stencil lies in the node's own 5 x 5 x 5 neighbourhood: the kernel sums that
// whole window with five weights per axis, one of them zero.  The addresses then depend on the node alone,
// and a row of the windows of four neighbours is eight consecutive floats, two 16-byte LDS reads per field.
//
// Why the window and not the 64 taps themselves: the taps start where the displacement puts them, so every
// tap of every node is its own LDS read (64 x 4 bytes per field, at the 128 bytes per clock and CU of reads
// below 16 bytes, plus a quarter more for bank conflicts), and those reads bounded the kernels: with the
// arithmetic taken out, the pair kernel at 128^3 kept 26 of its 28 us.  The window's reads
// are a sixth of that and run at the 256 bytes per clock of aligned 16-byte reads; its 125 products per field
// instead of 64 cost less than they free (a wave's FMA issues every two clocks).  At 128^3 (Infinity-Cache-resident
// fields), launches back to back: one field 19.6 -> 15.7 us, the adjoint pair 33.1 -> 23.5 us, three fields
// 48.0 -> 33.6 us; in a matvec, between other kernels: 21.2 -> 17.8, 31.8 -> 26.1; at 160x192x160 three fields
// 125 -> 75 us, the three components' pairs 198 -> 149 us.  What
// bounds it now is the window's arithmetic after a staging phase that a CU's two workgroups reach together
// (staging alone 11 us of the pair's 23.5, at 6.2 TB/s).
//
// Where one of a wave's nodes is displaced by a voxel or more, the wave sums the 64 taps of each of its nodes
// instead, from the brick where they lie in it, else from global memory, with the same products in the same
// order, so a node's value depends on neither the tile nor its neighbours.  Displacements of up to 1.5 voxels at
// 128^3: one field 26 us, the adjoint pair 40 us, three fields 60 us (the window and then the displaced nodes'
// taps: 49, 83 and 127 us; all nodes' taps always, in another layout: 34, 66 and 149 us); up to 10 voxels 102,
// 208 and 291 us (130, 218, 353; 114, 204, 368), bound by the gathers from global memory.
//
// The epilogue combines a node's interpolated values with its other pointwise operands, fusing the SL-RK2 step
// update of each equation into the same pass.
#include "kernels.h"

#include <climits>
#include <type_traits>
#include "prof.h"
#include "tune.h"

namespace lddmm {

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef const __attribute__((address_space(3))) float lds_float;
typedef __amdgpu_buffer_rsrc_t Rsrc;

constexpr int HALO = 2;

// Output tile of one workgroup; the autotuner picks one of these per grid shape and staging width.
// A row of the brick holds TX2 + 4 floats (a multiple of 16 bytes), fetched as QB aligned quads from two
// floats before it to two floats after it
template <int X0, int X1, int X2, int NT>
struct Tile {
  static constexpr int TX0 = X0, TX1 = X1, TX2 = X2, NTHR = NT;
  static constexpr int B0 = TX0 + 2 * HALO, B1 = TX1 + 2 * HALO, LD = TX2 + 2 * HALO;
  static constexpr int ROWS = B0 * B1, QB = TX2 / 4 + 2, NQ = ROWS * QB;
  static constexpr int VOL = ROWS * LD;               // LDS floats per field
  static constexpr int QPT = TX0 * TX1 * TX2 / 4 / NT;  // quads of nodes per thread
  static_assert(X2 % 4 == 0 && QPT * NT * 4 == TX0 * TX1 * TX2, "whole quads per thread");
};
using TileA = Tile<4, 8, 32, 256>;
using TileB = Tile<8, 8, 32, 512>;
using TileC = Tile<4, 4, 32, 128>;  // small grids: more workgroups
using TileD = Tile<4, 4, 64, 256>;
using TileE = Tile<8, 4, 32, 256>;
using TileF = Tile<4, 16, 32, 512>;
using TileG = Tile<8, 8, 16, 256>;  // a last tile of 16 on the contiguous axis
using TileH = Tile<4, 8, 64, 512>;
constexpr int kTiles = 8;

struct Grid3 {
  int n0, n1, n2;
  int64_t P;
};

__device__ __forceinline__ int wrapi(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}
// the same for indices that one period mostly brings back
__device__ __forceinline__ int wrap_near(int i, int n) {
  i = i < 0 ? i + n : i >= n ? i - n : i;
  if ((unsigned)i >= (unsigned)n) i = wrapi(i, n);
  return i;
}

// Cubic B-spline weights of the taps at -1, 0, 1, 2 for an offset t in [0, 1): (1-t)^3/6, 2/3 - t^2 (1 - t/2),
// the third from the partition of unity, t^3/6.
__device__ __forceinline__ void brick_weights(float t, float w[4]) {
  const float t2 = t * t, u = 1.f - t;
  w[3] = t2 * (t * (1.f / 6.f));
  w[0] = (u * u) * (u * (1.f / 6.f));
  w[1] = fmaf(t2, fmaf(t, 0.5f, -1.f), 2.f / 3.f);
  w[2] = 1.f - w[0] - w[1] - w[3];
}
// Weights of the five nodes at -2 .. 2 for a displacement d, |d| < 1: those of its fraction, from the node itself or
// the one before.  (Those of |d|, mirrored for d < 0, round the centre's weight up on both sides; over the steps of a
// state that sharpens an image's noise by 1e-6.)
__device__ __forceinline__ void window_weights(float d, float w[5]) {
  float v[4], t = d;
  const bool neg = d < 0.f;
  {
#pragma clang fp contract(off)  // not fused with the product that formed d: every tile rounds alike
    t = neg ? 1.f + d : d;
  }
  brick_weights(t, v);
  w[0] = neg ? v[0] : 0.f;
  w[1] = neg ? v[1] : v[0];
  w[2] = neg ? v[2] : v[1];
  w[3] = neg ? v[3] : v[2];
  w[4] = neg ? 0.f : v[3];
}

// Raw buffer accesses: 32-bit byte offsets from a uniform base, 0 for reads at or past the end
constexpr unsigned kOut = 0xFFFFFFF0u;
__device__ __forceinline__ Rsrc rsrc(const float* p, int64_t n) {
  const int64_t bytes = n * 4 < 0x7FFFFFF0 ? n * 4 : 0x7FFFFFF0;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float bload(Rsrc r, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ f32x4 bload4(Rsrc r, unsigned off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

// row sum of four taps, in the order of the window's (whose zero tap adds nothing)
__device__ __forceinline__ float row4(float a, float b, float c, float d, const float w[4]) {
  return fmaf(w[3], d, fmaf(w[2], c, fmaf(w[1], b, w[0] * a)));
}

// and of a node's own three
__device__ __forceinline__ float node3(float a, float b, float c) {
  return fmaf(1.f / 6.f, c, fmaf(2.f / 3.f, b, (1.f / 6.f) * a));
}

// p + n as a base that the compiler cannot see through, so that the reads around it take immediate offsets
__device__ __forceinline__ lds_float* opaque(lds_float* p, int n) {
  unsigned u = static_cast<unsigned>(reinterpret_cast<uintptr_t>(p + n));
  asm volatile("" : "+v"(u));
  return reinterpret_cast<lds_float*>(static_cast<uintptr_t>(u));
}

// periodic indices of the four taps around the node b
__device__ __forceinline__ void tap_nodes(int b, int n, int idx[4]) {
  b = wrapi(b, n);
  idx[0] = b == 0 ? n - 1 : b - 1;
#pragma unroll
  for (int o = 1; o < 4; ++o) idx[o] = idx[o - 1] + 1 == n ? 0 : idx[o - 1] + 1;
}

// 64-tap gather from global memory at the nodes (b0, b1, b2) plus the offsets t in [0, 1)
// (the grid sizes go by value: a reference would put the caller's Grid3 on the stack, a 24-byte
// scratch store per lane on every launch whether or not the gather runs)
__device__ __noinline__ float eval_global(const float* __restrict__ c, int b0, int b1, int b2, float t0, float t1,
                                          float t2, int n0, int n1, int n2) {
  int i0[4], i1[4], i2[4];
  float w0[4], w1[4], w2[4];
  tap_nodes(b0, n0, i0);
  tap_nodes(b1, n1, i1);
  tap_nodes(b2, n2, i2);
  brick_weights(t0, w0);
  brick_weights(t1, w1);
  brick_weights(t2, w2);
  float acc = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    float sa = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const float* row = c + (static_cast<int64_t>(i0[a]) * n1 + i1[b]) * n2;
      sa = fmaf(w1[b], row4(row[i2[0]], row[i2[1]], row[i2[2]], row[i2[3]], w2), sa);
    }
    acc = fmaf(w0[a], sa, acc);
  }
  return acc;
}

// Epilogues that also take the interpolant at the node itself
template <class E, class = void>
struct HasNode : std::false_type {};
template <class E>
struct HasNode<E, std::void_t<decltype(E::NODE)>> : std::bool_constant<E::NODE> {};

// Generic brick kernel.  Epi provides:
//   NF, FS       fields interpolated together and the stride between them (in fields) in `coef`;
//   NC           components launched together (component c's fields start at field c of `coef`);
//   NO           output fields (component c's results at field c of `out` when NC > 1);
//   struct In    a quad's operands; load(In&, rsrc of field k -> quad) reads them;
//   disp(In, k)  displacement of the four departure points along axis k (grid units);
//   finish(In, v, node, o)  results o[NO] from the interpolated values v[NF] (and the interpolants at the
//                nodes, node[NF], if NODE).
//   RAW: fields of less than 2^29 nodes, read by 32-bit byte offsets.
// Four waves a SIMD, so 128 registers: the single field and the pair take 97-106, three fields 120-128, of which the
// characteristics leave 2-3 in scratch (8 % more written; 35.3 us at 128^3, 37.5 before the wave took all its taps).
template <class Epi, class TL, bool RAW>
__global__ __launch_bounds__(TL::NTHR, 4) void k_brick(Epi epi, const float* __restrict__ coef, Grid3 g) {
  constexpr int TX0 = TL::TX0, TX1 = TL::TX1, TX2 = TL::TX2, NTHR = TL::NTHR, QPT = TL::QPT;
  constexpr int B0 = TL::B0, B1 = TL::B1, LD = TL::LD, QB = TL::QB, NQ = TL::NQ, VOL = TL::VOL;
  constexpr int NF = Epi::NF, NE = (NQ + NTHR - 1) / NTHR, Q2 = TX2 / 4;
  constexpr bool NODE = HasNode<Epi>::value;
  __shared__ __align__(16) float br[NF * VOL];
  // Workgroups are dealt to the 8 XCDs round-robin in launch order, so grid neighbours would sit in
  // different L2s and every halo would be fetched again from the fabric.  When the block count is a
  // multiple of 8 the launch index is remapped so that each XCD owns one contiguous run of tiles
  // (whole rows and slabs of the volume), whose shared halos then hit in its own L2.  The components of a
  // tile follow each other: they read the same displacements.
  const int gx = gridDim.x, gy = gridDim.y, nb = gx * gy * gridDim.z;
  int bid = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  if ((nb & 7) == 0) bid = (bid & 7) * (nb >> 3) + (bid >> 3);
  const int comp = bid % Epi::NC;
  bid /= Epi::NC;
  const int tx = gx / Epi::NC, bx = bid % tx, byz = bid / tx, by = byz % gy, bz = byz / gy;
  const int t0 = bz * TX0, t1 = by * TX1, t2 = bx * TX2;
  const int tid = threadIdx.x;
  const int64_t P = g.P, plane = (int64_t)g.n1 * g.n2;
  coef += comp * P;
  // staging: every load of the thread is requested before its first LDS store
  f32x4 v[NF][NE];
  Rsrc rs[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) rs[f] = rsrc(coef + f * Epi::FS * P, P);
#pragma unroll
  for (int k = 0; k < NE; ++k) {
    const int e = tid + k * NTHR;
    if (e < NQ) {
      const int row = e / QB, q = e - row * QB, b0 = row / B1, b1 = row - b0 * B1;
      const int r0 = wrap_near(t0 - HALO + b0, g.n0), r1 = wrap_near(t1 - HALO + b1, g.n1);
      const int c = wrap_near(t2 - 4 + 4 * q, g.n2);
      if constexpr (RAW) {
        const unsigned off = ((unsigned)(r0 * g.n1 + r1) * (unsigned)g.n2 + (unsigned)c) * 4u;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f][k] = bload4(rs[f], off);
        if (c + 3 >= g.n2) {  // the quad runs past the row's end (rows that are no multiple of four)
#pragma unroll
          for (int j = 1; j < 4; ++j) {
            const unsigned oj = off + 4u * (unsigned)(wrapi(c + j, g.n2) - c);
#pragma unroll
            for (int f = 0; f < NF; ++f) v[f][k][j] = bload(rs[f], oj);
          }
        }
      } else {
        const int64_t ro = ((int64_t)r0 * g.n1 + r1) * g.n2;
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
          for (int j = 0; j < 4; ++j) v[f][k][j] = coef[f * Epi::FS * P + ro + wrapi(c + j, g.n2)];
      }
    }
  }
  // pointwise operands of the thread's quads; offsets count from the tile's first plane
  typename Epi::In in[QPT];
  unsigned off[QPT];
  const int64_t base = t0 * plane, left = P - base;
#pragma unroll
  for (int j = 0; j < QPT; ++j) {
    const int q = tid + NTHR * j, l2 = (q % Q2) * 4, l1 = (q / Q2) % TX1, l0 = q / (Q2 * TX1);
    const int i0 = t0 + l0, i1 = t1 + l1, i2 = t2 + l2;
    const bool live = i0 < g.n0 && i1 < g.n1 && i2 < g.n2;
    off[j] = live ? ((unsigned)(l0 * g.n1 + i1) * (unsigned)g.n2 + (unsigned)i2) * 4u : kOut;
    epi.load(in[j], [&](const float* p) { return bload4(rsrc(p + base, left), off[j]); });
  }
#pragma unroll
  for (int k = 0; k < NE; ++k) {
    const int e = tid + k * NTHR;
    if (e < NQ) {
      const int row = e / QB, q = e - row * QB;
#pragma unroll
      for (int f = 0; f < NF; ++f) {  // a quad straddles the rows' two-float shift
        float* w = br + f * VOL + row * LD + 4 * q - 2;
        if (q > 0) *reinterpret_cast<f32x2*>(w) = f32x2{v[f][k].x, v[f][k].y};
        if (q < QB - 1) *reinterpret_cast<f32x2*>(w + 2) = f32x2{v[f][k].z, v[f][k].w};
      }
    }
  }
  __syncthreads();
  // The 64 taps of the tile's node (k0, k1, k2) displaced by (e0, e1, e2), from the brick if they lie in it, else from
  // global memory.  Where every lane's do, 4 x 4 taps of a field at a time, the next requested before the present are
  // summed; where some do not, a plane of taps at a time, whose sums all lanes share.
  auto taps = [&](int k0, int k1, int k2, float e0, float e1, float e2, float (&val)[NF]) {
    const float f0 = floorf(e0), f1 = floorf(e1), f2 = floorf(e2);
    float x0, x1, x2, u0[4], u1[4], u2[4];
    {
#pragma clang fp contract(off)  // not fused with the products that formed e, as in the window
      x0 = e0 - f0, x1 = e1 - f1, x2 = e2 - f2;
    }
    brick_weights(x0, u0);
    brick_weights(x1, u1);
    brick_weights(x2, u2);
    // (displacements beyond every grid are as good as none: the index is periodic)
    auto whole = [](float f) { return static_cast<int>(fabsf(f) < 1e9f ? f : 0.f); };
    const int d0 = whole(f0), d1 = whole(f1), d2 = whole(f2);
    // first tap in the brick
    const int s0 = k0 + HALO - 1 + d0, s1 = k1 + HALO - 1 + d1, s2 = k2 + HALO - 1 + d2;
    const bool inb = ((unsigned)s0 <= B0 - 4) & ((unsigned)s1 <= B1 - 4) & ((unsigned)s2 <= LD - 4);
    lds_float* p = (lds_float*)br + (inb ? (s0 * B1 + s1) * LD + s2 : 0);
#pragma unroll
    for (int f = 0; f < NF; ++f) val[f] = 0.f;
    auto read = [&](lds_float* r, float (&v)[4][4]) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[b][c] = r[b * LD + c];
    };
    auto sum = [&](const float (&v)[4][4]) {
      float sa = 0.f;
#pragma unroll
      for (int b = 0; b < 4; ++b) sa = fmaf(u1[b], row4(v[b][0], v[b][1], v[b][2], v[b][3], u2), sa);
      return sa;
    };
    if (__builtin_amdgcn_ballot_w64(!inb) == 0) {
      float d[2][4][4];
      read(opaque(p, 0), d[0]);
#pragma unroll
      for (int i = 0; i < 4 * NF; ++i) {
        if (i + 1 < 4 * NF) read(opaque(p, (i + 1) % NF * VOL + (i + 1) / NF * B1 * LD), d[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        val[i % NF] = fmaf(u0[i / NF], sum(d[i & 1]), val[i % NF]);
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    constexpr int FB = NF < 3 ? NF : 1;  // fields requested together, as the registers of four waves allow
    constexpr unsigned unit = RAW ? 4u : 1u;
    unsigned row[4] = {}, col[4] = {}, pl = 0;  // offsets of rows, columns and the plane
    int i0 = 0;
    if (!inb) {
      int i1[4], i2[4];
      i0 = wrapi(t0 + k0 + d0 % g.n0 - 1, g.n0);
      tap_nodes(t1 + k1 + d1 % g.n1, g.n1, i1);
      tap_nodes(t2 + k2 + d2 % g.n2, g.n2, i2);
      pl = (unsigned)i0 * (unsigned)plane * unit;
#pragma unroll
      for (int c = 0; c < 4; ++c) row[c] = (unsigned)i1[c] * (unsigned)g.n2 * unit, col[c] = (unsigned)i2[c] * unit;
    }
#pragma unroll 1
    for (int a = 0; a < 4; ++a) {
#pragma unroll
      for (int f0 = 0; f0 < NF; f0 += FB) {
        float v[FB][4][4];
#pragma unroll
        for (int f = 0; f < FB; ++f) read(p + (f0 + f) * VOL, v[f]);
        if (!inb) {
#pragma unroll
          for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(col[c]));  // (their 16 sums with the rows are not kept)
#pragma unroll
          for (int f = 0; f < FB; ++f)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if constexpr (RAW) v[f][b][c] = bload(rs[f0 + f], pl + row[b] + col[c]);
                else v[f][b][c] = coef[(f0 + f) * Epi::FS * P + (pl + row[b] + col[c])];
        }
#pragma unroll
        for (int f = 0; f < FB; ++f) val[f0 + f] = fmaf(u0[0], sum(v[f]), val[f0 + f]);
      }
      u0[0] = u0[1], u0[1] = u0[2], u0[2] = u0[3];
      if (inb) p += B1 * LD;
      pl += (unsigned)plane * unit;
      if (++i0 == g.n0) i0 = 0, pl = 0;
    }
  };
#pragma unroll
  for (int j = 0; j < QPT; ++j) {
    const int q = tid + NTHR * j, l2 = (q % Q2) * 4, l1 = (q / Q2) % TX1, l0 = q / (Q2 * TX1);
    bool far = false;  // a node displaced by a voxel or more
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const f32x4 d = epi.disp(in[j], k);
#pragma unroll
      for (int n = 0; n < 4; ++n) far |= !(fabsf(d[n]) < 1.f);
    }
    if (__builtin_amdgcn_ballot_w64(far) != 0) {
      // All taps (the window and the displaced nodes' taps after it take longer, see above), 64 neighbours of the
      // wave's 256 nodes at a time, a node a lane from its operands to its results: a tap of all lanes then lies in two
      // rows' lines and in as many banks as lanes (of the lanes' own quads, in eight rows' and a quarter of the banks).
      // The next nodes' operands are requested before the present taps.
      const int q0 = q - (tid & 63);
      auto place = [&](int n, int (&m)[3]) {
        const int e = 4 * q0 + 64 * n + (tid & 63);
        m[0] = e / (TX1 * TX2), m[1] = e / TX2 % TX1, m[2] = e % TX2;
        const int i1 = t1 + m[1], i2 = t2 + m[2];
        return t0 + m[0] < g.n0 && i1 < g.n1 && i2 < g.n2
                   ? ((unsigned)(m[0] * g.n1 + i1) * (unsigned)g.n2 + (unsigned)i2) * 4u : kOut;
      };
      typename Epi::In now, next;
      int m[3];
      unsigned at = place(0, m);
      auto fetch = [&](typename Epi::In& x, unsigned o) {
        epi.load(x, [&](const float* p) { return f32x4{bload(rsrc(p + base, left), o), 0.f, 0.f, 0.f}; });
      };
      fetch(now, at);
#pragma unroll 1
      for (int n = 0; n < 4; ++n) {
        int mn[3];
        const unsigned an = place(n + 1, mn);
        if (n < 3) fetch(next, an);
        float val[NF];
        taps(m[0], m[1], m[2], epi.disp(now, 0).x, epi.disp(now, 1).x, epi.disp(now, 2).x, val);
        f32x4 v[NF], nv[NF], o[Epi::NO];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          v[f] = f32x4{val[f], 0.f, 0.f, 0.f}, nv[f] = f32x4{0.f, 0.f, 0.f, 0.f};
          if constexpr (NODE) {
            lds_float* p = (lds_float*)br + f * VOL + ((m[0] + HALO) * B1 + m[1] + HALO) * LD + m[2] + HALO;
#pragma unroll
            for (int a = -1; a < 2; ++a) {
              float sn = 0.f;
#pragma unroll
              for (int b = -1; b < 2; ++b) {
                lds_float* r = p + (a * B1 + b) * LD;
                sn = fmaf(b == 0 ? 2.f / 3.f : 1.f / 6.f, node3(r[-1], r[0], r[1]), sn);
              }
              nv[f].x = fmaf(a == 0 ? 2.f / 3.f : 1.f / 6.f, sn, nv[f].x);
            }
          }
        }
        epi.finish(now, v, nv, o);
#pragma unroll
        for (int k = 0; k < Epi::NO; ++k)
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)o[k].x),
                                                rsrc(epi.out + (comp + k) * P + base, left), (int)at, 0, 0);
        now = next, at = an;
#pragma unroll
        for (int k = 0; k < 3; ++k) m[k] = mn[k];
      }
      continue;
    }
    float w0[4][5], w1[4][5], w2[4][5];
    {
      const f32x4 d0 = epi.disp(in[j], 0), d1 = epi.disp(in[j], 1), d2 = epi.disp(in[j], 2);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        window_weights(d0[n], w0[n]);
        window_weights(d1[n], w1[n]);
        window_weights(d2[n], w2[n]);
      }
    }
    f32x4 acc[NF], node[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = node[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float* win = br + (l0 * B1 + l1) * LD + l2;
#pragma unroll 1
    for (int a = 0; a < 5; ++a) {
      f32x4 s[NF], sn[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) s[f] = sn[f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int b = 0; b < 5; ++b) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          lds_f32x4* p = (lds_f32x4*)((lds_float*)win + f * VOL + (a * B1 + b) * LD);
          const f32x4 lo = p[0], hi = p[1];
          const float r[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          float t[4];
#pragma unroll
          for (int n = 0; n < 4; ++n) t[n] = w2[n][0] * r[n];
#pragma unroll
          for (int c = 1; c < 5; ++c)
#pragma unroll
            for (int n = 0; n < 4; ++n) t[n] = fmaf(w2[n][c], r[n + c], t[n]);
#pragma unroll
          for (int n = 0; n < 4; ++n) s[f][n] = fmaf(w1[n][b], t[n], s[f][n]);
          // (three fields' rows are not all requested at once: 184 registers in the tiles of few threads)
          if constexpr (NF >= 3 && !NODE)
            if (f == NF - 1 && b % 2) __builtin_amdgcn_sched_barrier(0);
          if constexpr (NODE) {  // taps (1/6, 2/3, 1/6) around the node
            if (b >= 1 && b <= 3) {
              const float wb = b == 2 ? 2.f / 3.f : 1.f / 6.f;
#pragma unroll
              for (int n = 0; n < 4; ++n)
                sn[f][n] = fmaf(wb, node3(r[n + 1], r[n + 2], r[n + 3]), sn[f][n]);
            }
          }
        }
      }
      const float wa = a == 2 ? 2.f / 3.f : (a == 1 || a == 3) ? 1.f / 6.f : 0.f;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const float w = w0[n][0];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          acc[f][n] = fmaf(w, s[f][n], acc[f][n]);
          if constexpr (NODE) node[f][n] = fmaf(wa, sn[f][n], node[f][n]);
        }
        w0[n][0] = w0[n][1], w0[n][1] = w0[n][2], w0[n][2] = w0[n][3], w0[n][3] = w0[n][4];
      }
    }
    if (off[j] == kOut) continue;
    f32x4 o[Epi::NO];
    epi.finish(in[j], acc, node, o);
    const int last = g.n2 - (t2 + l2);  // nodes left in the row
#pragma unroll
    for (int k = 0; k < Epi::NO; ++k) {
      const Rsrc ro = rsrc(epi.out + (comp + k) * P + base, left);
      typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
      if (last >= 4) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[k]), ro, (int)off[j], 0, 0);
      } else {
#pragma unroll
        for (int n = 0; n < 3; ++n) {
          const float w = o[k][n];  // (a scalar of its own: a bit cast of a vector element takes element 0)
          if (n < last)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, w), ro, (int)(off[j] + 4u * n), 0, 0);
        }
      }
    }
  }
}

// ---- epilogues ---------------------------------------------------------------------

template <int NFv, int FSv = 1, int NCv = 1, int NOv = NFv>
struct Shape {
  static constexpr int NF = NFv, FS = FSv, NC = NCv, NO = NOv;
};

// nodes displaced by a stored departure displacement field (grid units)
struct Displaced {
  const float* __restrict__ dsp;
  int64_t P;
  struct In {
    f32x4 d[3];
  };
  template <class L>
  __device__ __forceinline__ void load(In& in, L&& ld) const {
#pragma unroll
    for (int k = 0; k < 3; ++k) in.d[k] = ld(dsp + k * P);
  }
  __device__ __forceinline__ f32x4 disp(const In& in, int k) const { return in.d[k]; }
};
// the same with the velocity divergence at the node
struct DisplacedDiv : Displaced {
  const float* __restrict__ divv;
  struct In : Displaced::In {
    f32x4 v;
  };
  template <class L>
  __device__ __forceinline__ void load(In& in, L&& ld) const {
    Displaced::load(in, ld);
    in.v = ld(divv);
  }
  __device__ __forceinline__ f32x4 disp(const In& in, int k) const { return in.d[k]; }
};

template <int NFv>
struct EpiInterp : Displaced, Shape<NFv> {
  float* __restrict__ out;
  __device__ __forceinline__ void finish(const In&, const f32x4* v, const f32x4*, f32x4* o) const {
#pragma unroll
    for (int f = 0; f < NFv; ++f) o[f] = v[f];
  }
};

// out_f = P(c_f) o X - P(c_f)(x): the interpolant's change along the characteristic (projected, it is
// the step's increment of a band-limited field, whose own projection the caller adds back exactly)
template <int NFv>
struct EpiInterpDiff : Displaced, Shape<NFv> {
  static constexpr bool NODE = true;
  float* __restrict__ out;
  __device__ __forceinline__ void finish(const In&, const f32x4* v, const f32x4* node, f32x4* o) const {
#pragma unroll
    for (int f = 0; f < NFv; ++f) o[f] = v[f] - node[f];
  }
};

// band-limited adjoint Heun step of NCv components (one per workgroup): out_c = cA_c o X + dt/2 divv (cB_c o X),
// fields [cA_0 .. cA_{NCv-1}, cB_0 .. cB_{NCv-1}]
template <int NCv>
struct EpiBLAdjoint : DisplacedDiv, Shape<2, NCv, NCv, 1> {
  float* __restrict__ out;
  float dt;
  __device__ __forceinline__ void finish(const In& in, const f32x4* v, const f32x4*, f32x4* o) const {
#pragma unroll
    for (int n = 0; n < 4; ++n) o[0][n] = v[0][n] + 0.5f * dt * in.v[n] * v[1][n];
  }
};

// image-transport adjoint on the grid: a = c1 o X, b = c2 o X,
// out = a + dt/2 (b + (a + dt b) divv) = (1 + dt/2 divv) a + dt/2 (1 + dt divv) b
struct EpiAdjointGrid : DisplacedDiv, Shape<2, 1, 1, 1> {
  float* __restrict__ out;
  float dt;
  __device__ __forceinline__ void finish(const In& in, const f32x4* v, const f32x4*, f32x4* o) const {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const float dv = in.v[n];
      o[0][n] = (1.f + 0.5f * dt * dv) * v[0][n] + 0.5f * dt * (1.f + dt * dv) * v[1][n];
    }
  }
};

// characteristics: X* = x + sdt v, X - x = sdt/2 (v + v o X*) (grid units)
struct EpiCharacteristics : Shape<3> {
  const float* __restrict__ v;
  float* __restrict__ out;
  int64_t P;
  float sdt, s0, s1, s2;  // signed dt and per-axis grid sizes
  struct In {
    f32x4 v[3];
  };
  template <class L>
  __device__ __forceinline__ void load(In& in, L&& ld) const {
#pragma unroll
    for (int k = 0; k < 3; ++k) in.v[k] = ld(v + k * P);
  }
  __device__ __forceinline__ float scale(int k) const { return k == 0 ? s0 : k == 1 ? s1 : s2; }
  __device__ __forceinline__ f32x4 disp(const In& in, int k) const {
    f32x4 d;
#pragma unroll
    for (int n = 0; n < 4; ++n) d[n] = sdt * in.v[k][n] * scale(k);
    return d;
  }
  __device__ __forceinline__ void finish(const In& in, const f32x4* c, const f32x4*, f32x4* o) const {
    const float h = 0.5f * sdt;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int n = 0; n < 4; ++n) o[k][n] = h * (in.v[k][n] * scale(k) + c[k][n] * scale(k));
  }
};

template <class Epi, class TL, bool RAW = true>
void launch_tile(const std::string& name, double bytes, const Epi& epi, const float* coef, const Grid3& g,
                 hipStream_t s) {
  dim3 grid(ceil_div(g.n2, TL::TX2) * Epi::NC, ceil_div(g.n1, TL::TX1), ceil_div(g.n0, TL::TX0));
  prof::launch(name, bytes, 0.0, k_brick<Epi, TL, RAW>, grid, dim3(TL::NTHR), 0, s, epi, coef, g);
}

std::string shape_key(const Dims& d) {
  return "brick:" + std::to_string(d.n[0]) + "x" + std::to_string(d.n[1]) + "x" + std::to_string(d.n[2]);
}

template <class Epi>
void launch(const std::string& name, double bytes, const Epi& epi, const float* coef, const Dims& d,
            hipStream_t s, int tile = -1) {
  const Grid3 g{d.n[0], d.n[1], d.n[2], d.P};
  if (d.P >= (int64_t(1) << 29)) {
    launch_tile<Epi, TileA, false>(name, bytes, epi, coef, g, s);
    LDDMM_LAUNCH_CHECK();
    return;
  }
  if (tile < 0) tile = std::max(0, tune::get(shape_key(d) + ":gs" + std::to_string(Epi::NF), 0));
  switch (tile) {
    case 1:
      launch_tile<Epi, TileB>(name, bytes, epi, coef, g, s);
      break;
    case 2:
      launch_tile<Epi, TileC>(name, bytes, epi, coef, g, s);
      break;
    case 3:
      launch_tile<Epi, TileD>(name, bytes, epi, coef, g, s);
      break;
    case 4:
      launch_tile<Epi, TileE>(name, bytes, epi, coef, g, s);
      break;
    case 5:
      launch_tile<Epi, TileF>(name, bytes, epi, coef, g, s);
      break;
    case 6:
      launch_tile<Epi, TileG>(name, bytes, epi, coef, g, s);
      break;
    case 7:
      launch_tile<Epi, TileH>(name, bytes, epi, coef, g, s);
      break;
    default:
      launch_tile<Epi, TileA>(name, bytes, epi, coef, g, s);
  }
  LDDMM_LAUNCH_CHECK();
}

std::string nm(const char* base) { return std::string("k_brick<") + base + ">"; }

// smooth sub-voxel departure displacements (amplitude 0.8 voxel) for timing the tiles under the
// LDS access pattern of real steps
__global__ void k_tune_disp(float* disp, int n0, int n1, int n2) {
  const int64_t P = (int64_t)n0 * n1 * n2;
  const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (p >= P) return;
  const int i2 = (int)(p % n2), i1 = (int)((p / n2) % n1), i0 = (int)(p / ((int64_t)n1 * n2));
  const float ph = 6.2831853f * ((float)i0 / n0 + 2.f * i1 / n1 + 3.f * i2 / n2);
#pragma unroll
  for (int c = 0; c < 3; ++c) disp[c * P + p] = 0.8f * sinf(ph + 1.7f * c);
}

// ---- transformation through whole-deformation maps ------------------------------------

// 64-tap evaluation from a staged box of planes of `plane` floats and rows of `pitch`, first tap at br
__device__ __forceinline__ float eval_box(lds_float* br, int plane, int pitch, const float w0[4], const float w1[4],
                                          const float w2[4]) {
  float acc = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    float sa = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      lds_float* row = br + (a * plane + b * pitch);
      sa += w1[b] * (w2[0] * row[0] + w2[1] * row[1] + w2[2] * row[2] + w2[3] * row[3]);
    }
    acc += w0[a] * sa;
  }
  return acc;
}

// out_n(x) = a w_n(x) P(c)(x - u_n(x)) for node n = blockIdx.y (u_n [3][P] in unit-torus units, w_n
// optional).  The departure points lie up to a whole deformation away from their nodes, beyond any
// fixed halo, but they move smoothly: the workgroup takes the bounding box of its tile's 4 x 4 x 4
// stencils, stages the box into LDS when it holds at most CAP floats and evaluates every node from
// there; a larger box falls back to gathers from global memory.  Three phases wait for each other
// (displacements, box, taps), so each is kept short: bounds are packed 16-bit pairs reduced by shuffles,
// a thread requests its share of the box (some ten values, walked without divisions) at once, and rows
// keep a pitch of 8 modulo 16, which spreads the four tile rows of a wave over the banks.  Eleven nodes
// of 128^3: 650 -> 338 us (31 us a node, 42 MB; 1024 threads 530, tiles of 4 x 8 x 16 397, of 8 x 8 x 32 633).
template <int TX0, int TX1, int TX2, int NTHR, int CAP>
__global__ __launch_bounds__(NTHR) void k_pull_back_box(float* __restrict__ out, const float* __restrict__ c,
                                                        const float* __restrict__ u, const float* __restrict__ w,
                                                        float a, Grid3 g) {
  constexpr int PPT = TX0 * TX1 * TX2 / NTHR, NW = NTHR / 64, U = 12;
  typedef short s16x2 __attribute__((ext_vector_type(2)));
  __shared__ float br[CAP];
  __shared__ int bounds[NW][3];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T2 = (g.n2 + TX2 - 1) / TX2, T1 = (g.n1 + TX1 - 1) / TX1;
  // consecutive tiles of one node on one XCD (its L2 then holds the boxes' overlap)
  const int nb = gridDim.x;
  int bid = blockIdx.x;
  if ((nb & 7) == 0) bid = (bid & 7) * (nb >> 3) + (bid >> 3);
  const int bx = bid % T2, rest = bid / T2, by = rest % T1, bz = rest / T1;
  const int org[3] = {bz * TX0, by * TX1, bx * TX2};
  const int64_t P = g.P, node = blockIdx.y;
  const float* __restrict__ un = u + node * 3 * P;
  const float* __restrict__ wn = w ? w + node * P : nullptr;
  float x[PPT][3], fac[PPT];
  int pidx[PPT];
  bool live[PPT];
#pragma unroll
  for (int j = 0; j < PPT; ++j) {
    const int q = tid + NTHR * j;
    const int i0 = org[0] + q / (TX1 * TX2), i1 = org[1] + (q / TX2) % TX1, i2 = org[2] + q % TX2;
    live[j] = i0 < g.n0 && i1 < g.n1 && i2 < g.n2;
    pidx[j] = live[j] ? (i0 * g.n1 + i1) * g.n2 + i2 : 0;
    x[j][0] = un[pidx[j]], x[j][1] = un[P + pidx[j]], x[j][2] = un[2 * P + pidx[j]];
    fac[j] = wn ? wn[pidx[j]] : 1.f;
  }
  // bounds of the stencils relative to the tile, (min, -max) per axis; 16 bits hold any box worth staging
  s16x2 bnd[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) bnd[k] = s16x2{16000, 16000};
#pragma unroll
  for (int j = 0; j < PPT; ++j) {
    const int q = tid + NTHR * j;
    const int n[3] = {g.n0, g.n1, g.n2}, l[3] = {q / (TX1 * TX2), (q / TX2) % TX1, q % TX2};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      x[j][k] = (org[k] + l[k]) - x[j][k] * n[k];
      const short f = static_cast<short>(fminf(fmaxf(floorf(x[j][k]) - org[k], -15000.f), 15000.f));
      if (live[j]) bnd[k] = __builtin_elementwise_min(bnd[k], s16x2{(short)(f - 1), (short)(-f - 2)});
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
      bnd[k] = __builtin_elementwise_min(
          bnd[k], __builtin_bit_cast(s16x2, __shfl_xor(__builtin_bit_cast(int, bnd[k]), o)));
    if (lane == 0) bounds[wave][k] = __builtin_bit_cast(int, bnd[k]);
  }
  __syncthreads();
  int lo[3], e[3];
  bool near = true;  // no bound was clamped (nor a point NaN)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s16x2 b = __builtin_bit_cast(s16x2, bounds[0][k]);
#pragma unroll
    for (int v = 1; v < NW; ++v) b = __builtin_elementwise_min(b, __builtin_bit_cast(s16x2, bounds[v][k]));
    lo[k] = __builtin_amdgcn_readfirstlane(b[0] + org[k]);
    e[k] = __builtin_amdgcn_readfirstlane(1 - b[0] - b[1]);
    near = near && b[0] > -14000 && b[1] > -14000;
  }
  // (every tile holds a live node, the grid is ceil-divided: e >= 4)
  const int pitch = ((e[2] + 7) & ~15) + 8, plane = e[1] * pitch;
  const bool staged = near && e[0] <= g.n0 && e[1] <= g.n1 && e[2] <= g.n2 && (int64_t)e[0] * plane <= CAP;
  if (staged) {
    const int m0 = wrapi(lo[0], g.n0), m1 = wrapi(lo[1], g.n1), m2 = wrapi(lo[2], g.n2);
    const int total = e[0] * e[1] * e[2];
    // element tid, tid + NTHR, ..: (r0, r1, col) advanced by the step's digits
    const int dr = NTHR / e[2], d2 = NTHR - dr * e[2], d0 = dr / e[1], d1 = dr - d0 * e[1];
    int col = tid % e[2], r1 = tid / e[2], r0 = r1 / e[1];
    r1 -= r0 * e[1];
    for (int t0 = tid; t0 < total; t0 += NTHR * U) {
      float v[U];
      int at[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        int y0 = m0 + r0, y1 = m1 + r1, y2 = m2 + col;
        y0 = y0 >= g.n0 ? y0 - g.n0 : y0;
        y1 = y1 >= g.n1 ? y1 - g.n1 : y1;
        y2 = y2 >= g.n2 ? y2 - g.n2 : y2;
        const bool ok = t0 + NTHR * k < total;
        at[k] = ok ? r0 * plane + r1 * pitch + col : -1;
        v[k] = c[ok ? (y0 * g.n1 + y1) * g.n2 + y2 : 0];
        col += d2, r1 += d1, r0 += d0;
        if (col >= e[2]) col -= e[2], ++r1;
        if (r1 >= e[1]) r1 -= e[1], ++r0;
      }
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (at[k] >= 0) br[at[k]] = v[k];
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < PPT; ++j) {
    if (!live[j]) continue;
    const float f0 = floorf(x[j][0]), f1 = floorf(x[j][1]), f2 = floorf(x[j][2]);
    float val;
    if (staged) {
      float w0[4], w1[4], w2[4];
      bspline_weights(x[j][0] - f0, w0);
      bspline_weights(x[j][1] - f1, w1);
      bspline_weights(x[j][2] - f2, w2);
      const int s0 = static_cast<int>(f0) - 1 - lo[0], s1 = static_cast<int>(f1) - 1 - lo[1],
                s2 = static_cast<int>(f2) - 1 - lo[2];
      val = eval_box((lds_float*)br + (s0 * plane + s1 * pitch + s2), plane, pitch, w0, w1, w2);
    } else {
      val = eval_global(c, static_cast<int>(f0), static_cast<int>(f1), static_cast<int>(f2), x[j][0] - f0, x[j][1] - f1,
                        x[j][2] - f2, g.n0, g.n1, g.n2);
    }
    out[node * P + pidx[j]] = a * (w ? fac[j] * val : val);
  }
}

}  // namespace

bool brick_ok(const Dims& d) { return d.n[0] > 1; }

void brick_pull_back(float* out, const float* c, const float* u, const float* w, float a, int nodes, const Dims& d,
                     hipStream_t s) {
  // 8 x 8 x 16 nodes per workgroup: the boxes of an 8-voxel deformation of 128^3 hold 5 staged values per
  // node on average and all fit in 8192 floats (32 KB, four workgroups of eight waves per CU)
  constexpr int TX0 = 8, TX1 = 8, TX2 = 16, NTHR = 512, CAP = 8192;
  if (nodes < 1 || nodes > 65535) throw ArgError("brick_pull_back: node count out of range");
  const Grid3 g{d.n[0], d.n[1], d.n[2], d.P};
  const int64_t tiles = (int64_t)ceil_div(d.n[0], TX0) * ceil_div(d.n[1], TX1) * ceil_div(d.n[2], TX2);
  if (tiles > INT_MAX) throw ArgError("brick_pull_back: grid too large");
  prof::launch("k_pull_back_box", double(nodes) * (w ? 5.0 : 4.0) * d.P * 4 + d.P * 4.0, 0.0,
               k_pull_back_box<TX0, TX1, TX2, NTHR, CAP>, dim3(static_cast<unsigned>(tiles), nodes), dim3(NTHR), 0,
               s, out, c, u, w, a, g);
  LDDMM_LAUNCH_CHECK();
}

int brick_tile_count() { return kTiles; }

// One tile per grid shape and staging width (fields staged together: 1, 2 or 3), timed on the epilogues of
// that width that the sweeps launch most (the pair: one component's adjoint step); out holds 3 fields, coef 3
// fields.
void brick_autotune(float* out, const float* coef, float* disp, const Dims& d, hipStream_t s) {
  const std::string key = shape_key(d) + ":gs";
  if (tune::get(key + "1", -1) >= 0 && tune::get(key + "2", -1) >= 0 && tune::get(key + "3", -1) >= 0) return;
  k_tune_disp<<<ceil_div(d.P, 256), 256, 0, s>>>(disp, d.n[0], d.n[1], d.n[2]);
  LDDMM_LAUNCH_CHECK();
  EpiInterp<1> e1;
  e1.dsp = disp, e1.P = d.P, e1.out = out;
  EpiBLAdjoint<1> e2;
  e2.dsp = disp, e2.P = d.P, e2.out = out, e2.divv = coef + 2 * d.P, e2.dt = 0.1f;
  EpiInterp<3> e3;
  e3.dsp = disp, e3.P = d.P, e3.out = out;
  tune::set(key + "1", tune::pick(kTiles, [&](int c) { launch("tune", 0.0, e1, coef, d, s, c); }, s));
  tune::set(key + "2", tune::pick(kTiles, [&](int c) { launch("tune", 0.0, e2, coef, d, s, c); }, s));
  tune::set(key + "3", tune::pick(kTiles, [&](int c) { launch("tune", 0.0, e3, coef, d, s, c); }, s));
}

template <template <int> class Epi>
static void interp_any(const char* base, float* out, const float* coef, int nf, const float* disp, const Dims& d,
                       hipStream_t s) {
  const std::string name_ = nm(base) + std::to_string(nf);
  const double bytes_ = (3.0 + 2.0 * nf) * d.P * 4;
  if (nf == 1) {
    Epi<1> e;
    e.dsp = disp, e.P = d.P, e.out = out;
    launch(name_, bytes_, e, coef, d, s);
  } else if (nf == 3) {
    Epi<3> e;
    e.dsp = disp, e.P = d.P, e.out = out;
    launch(name_, bytes_, e, coef, d, s);
  } else {
    throw ArgError(std::string(base) + ": nf must be 1 or 3");
  }
}

void brick_interp(float* out, const float* coef, int nf, const float* disp, const Dims& d, hipStream_t s) {
  interp_any<EpiInterp>("k_interp", out, coef, nf, disp, d, s);
}

void brick_interp_diff(float* out, const float* coef, int nf, const float* disp, const Dims& d, hipStream_t s) {
  interp_any<EpiInterpDiff>("k_interp_diff", out, coef, nf, disp, d, s);
}

void brick_bl_adjoint_step(float* out, const float* cAB, int nc, const float* disp, const float* divv,
                           const Dims& d, float dt, hipStream_t s) {
  const std::string name_ = nm("k_bl_adjoint_step") + std::to_string(nc);
  const double bytes_ = (4.0 + 3.0 * nc) * d.P * 4;
  auto go = [&](auto e) {
    e.dsp = disp, e.P = d.P, e.out = out, e.divv = divv, e.dt = dt;
    launch(name_, bytes_, e, cAB, d, s);
  };
  // three components: one workgroup per component and tile on its pair (cA_c, cB_c), which keeps the registers
  // (and the occupancy) of the one-component kernel; in one launch, so that the components of a tile share
  // its displacements in the caches
  if (nc == 1) go(EpiBLAdjoint<1>{});
  else if (nc == 3) go(EpiBLAdjoint<3>{});
  else throw ArgError("brick_bl_adjoint_step: nc must be 1 or 3");
}

void brick_adjoint_grid_step(float* out, const float* c12, const float* disp, const float* divv, const Dims& d,
                             float dt, hipStream_t s) {
  const std::string name_ = nm("k_adjoint_grid_step");
  const double bytes_ = 7.0 * d.P * 4;
  EpiAdjointGrid e;
  e.dsp = disp, e.P = d.P, e.out = out, e.divv = divv, e.dt = dt;
  launch(name_, bytes_, e, c12, d, s);
}

void brick_characteristics(float* disp, const float* v, const float* cv, const Dims& d, float dt, int dir,
                           hipStream_t s) {
  const std::string name_ = nm("k_characteristics");
  const double bytes_ = 9.0 * d.P * 4;
  EpiCharacteristics e;
  e.v = v, e.out = disp, e.P = d.P;
  e.sdt = dir > 0 ? dt : -dt;
  e.s0 = float(d.n[0]), e.s1 = float(d.n[1]), e.s2 = float(d.n[2]);
  launch(name_, bytes_, e, cv, d, s);
}

}  // namespace lddmm
