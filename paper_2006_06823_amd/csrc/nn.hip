// Learned warm start and low-rank PCG preconditioner: a small 3D convolutional
// encoder with hand-written bf16 matrix-core kernels (forward, backward-data,
// backward-weight), float master weights and Adam, all on the device.
//
// Convolutions are implicit GEMMs on v_mfma_f32_32x32x16_bf16 (operands rounded to
// bf16, float accumulation):
//   forward      Y[b][co][o]       = act(bias[co] + sum_{ci,t} W[co][ci][t] X[b][ci][pos(o,t)])
//   backward-data dX[b][ci][i]     = sum_{co,t} W[co][ci][t] G[b][co][o(i,t)]   (o(i,t) when it exists)
//   backward-wt   dW[co][ci][t]   += sum_{b,o} G[b][co][o] X[b][ci][pos(o,t)]  (split over blocks)
// with G = dY * act'(Y).  Activations are [B][C][D][H][W] float.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <type_traits>
#include <vector>

#include "nn.h"
#include "prof.h"

namespace lddmm {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

namespace {

__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

__device__ __forceinline__ unsigned short bf16_rn(float x) {
  const unsigned int b = __float_as_uint(x);
  return static_cast<unsigned short>((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ bf16x8 to_bf16x8(const float v[8]) {
  u16x8 h;
#pragma unroll
  for (int j = 0; j < 8; ++j) h[j] = bf16_rn(v[j]);
  return __builtin_bit_cast(bf16x8, h);
}

// ---- convolutions -----------------------------------------------------------------------------
// One kernel serves the forward pass and the data gradient: both are convolutions of a "virtual" input
// (forward: x; data gradient: G with zeros between its samples where the layer has a stride) at every
// output position.  A workgroup owns a box of 128 output voxels (32 per wave) of one sample and MT tiles
// of 32 output channels.  It converts the box's input patch (the box plus the kernel's halo, 16 channels
// at a time) to bf16 once, into LDS; a lane then gathers the eight bf16 operands of a k-step from there
// with one add each (the offsets of the 16 x k^3 steps of a channel group are tabulated in LDS), and the
// fragment serves the MT channel tiles.  The weights come packed in fragment order, one 16-byte load per
// lane and tile.  The k-steps follow the flattened (channel, tap) index, 16 per matrix instruction, so the
// sums are independent of box and tile.  What bounds it: the gathers (8 LDS reads and 8 adds per k-step
// against MT matrix instructions of 32 cycles); patch, packed weights and MT remove the repeated index
// arithmetic, conversions and L2 reads of a gather straight from global memory.  Batch 16 of 64^3
// pairs through 2-16-32-64-128-3 channels, against that gather: forward 1.60 -> 0.18 ms, data gradient
// 4.29 -> 0.19 ms (64 -> 128 channels at 16^3, 29 GFLOP: 61 and 69 us, 0.48 and 0.42 PFLOP/s).
struct ConvArgs {
  const void* in;            // forward: x [B][Cin][Di^3] float; data gradient: G [B][Cin][Di^3] bf16
  const unsigned short* ap;  // packed weights [M / 32][chunks][64][8] (bf16)
  const float* b;            // bias (forward)
  float* y;                  // [B][M][No^3]
  int Cin, M, Di, Do;        // channels contracted, output channels, input and output edge
  int pad, up, relu;         // halo before the first tap; zero-insertion factor of the virtual input
  int nb;                    // boxes per sample
};

// Box shapes of 128 voxels; the host takes the one that wastes least of an edge
template <int X, int Y, int Z>
struct Box {
  static constexpr int BX = X, BY = Y, BZ = Z;
  static_assert(X * Y * Z == 128, "four waves of 32 voxels");
};
using BoxWide = Box<32, 4, 1>;
using BoxMid = Box<16, 4, 2>;
using BoxSmall = Box<8, 4, 4>;

template <class BoxT, int KS, int S>
struct Patch {
  static constexpr int PX = (BoxT::BX - 1) * S + KS, PY = (BoxT::BY - 1) * S + KS, PZ = (BoxT::BZ - 1) * S + KS;
  static constexpr int PV = PX * PY * PZ;
  static constexpr int TP = PV > 128 ? 256 : 128;      // threads across the positions (the others: channels)
  static constexpr int NPOS = (PV + TP - 1) / TP;      // positions per thread
};

// Raw buffer loads: an offset register per position and the channel's base in scalar registers, no address
// arithmetic per value; the range check returns 0 for kOut, so padding needs no select.  Offsets count from
// the first plane of a patch (they fit 32 bits for every grid).
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr unsigned kOut = 0xFFFFFFF0u;
template <typename T>
__device__ __forceinline__ Rsrc rsrc(const T* p, int64_t n) {
  const int64_t bytes = n * (int64_t)sizeof(T) < 0x7FFFFFF0 ? n * (int64_t)sizeof(T) : 0x7FFFFFF0;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float bload_f(Rsrc r, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ unsigned short bload_h(Rsrc r, unsigned off) {
  return __builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
}

template <class BoxT>
__device__ __forceinline__ void box_origin(int box, int D, int o[3]) {
  const int nx = (D + BoxT::BX - 1) / BoxT::BX, ny = (D + BoxT::BY - 1) / BoxT::BY;
  const int bx = box % nx, r = box / nx, by = r % ny, bz = r / ny;
  o[0] = bz * BoxT::BZ, o[1] = by * BoxT::BY, o[2] = bx * BoxT::BX;
}

template <class BoxT, int KS, int S, int MT, bool BWD>
__global__ __launch_bounds__(256) void k_conv(ConvArgs a) {
  using P = Patch<BoxT, KS, S>;
  constexpr int K3 = KS * KS * KS, CG = KS == 3 ? 16 : 64, KG = CG * K3;  // channels and k-steps of a group
  constexpr int PD = KS == 3 ? 3 : 2;  // chunks of weights in flight (a full group is a multiple of them)
  __shared__ unsigned short patch[CG * P::PV];
  __shared__ __align__(16) unsigned tab[KG];  // element offset of each k-step of a group in the patch
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 31, kh = lane >> 5;
  const int D = a.Di, Do = a.Do;
  const int64_t Ni = (int64_t)D * D * D, No = (int64_t)Do * Do * Do;
  const int b = blockIdx.z, m0 = blockIdx.y * 32 * MT;
  int o0[3];
  box_origin<BoxT>(blockIdx.x, Do, o0);
  for (int k = tid; k < KG; k += 256) {
    const int c = k / K3, t = k - c * K3, tz = t / (KS * KS), ty = (t / KS) % KS, tx = t % KS;
    // the data gradient meets tap t at u = i + pad - t: the patch read backwards
    const int z = BWD ? KS - 1 - tz : tz, y = BWD ? KS - 1 - ty : ty, x = BWD ? KS - 1 - tx : tx;
    tab[k] = (unsigned)(c * P::PV + (z * P::PY + y) * P::PX + x);
  }
  using In = std::conditional_t<BWD, unsigned short, float>;
  constexpr unsigned ES = sizeof(In);
  const int before = BWD ? KS - 1 - a.pad : a.pad;
  // first input plane the patch can reach, and byte offset from it (kOut: padding) of each staged position
  const int z0 = o0[0] * S - before, zlo = z0 <= 0 ? 0 : BWD ? z0 / a.up : z0;
  unsigned pos[P::NPOS];
#pragma unroll
  for (int i = 0; i < P::NPOS; ++i) {
    const int e = tid % P::TP + P::TP * i;
    const int x = e % P::PX, y = (e / P::PX) % P::PY, z = e / (P::PX * P::PY);
    int u0 = z0 + z, u1 = o0[1] * S + y - before, u2 = o0[2] * S + x - before;
    bool ok = e < P::PV && u0 >= 0 && u1 >= 0 && u2 >= 0;
    if (BWD && a.up > 1) {
      ok = ok && u0 % a.up == 0 && u1 % a.up == 0 && u2 % a.up == 0;
      u0 /= a.up, u1 /= a.up, u2 /= a.up;
    }
    ok = ok && u0 < D && u1 < D && u2 < D;
    pos[i] = ok ? (unsigned)(((u0 - zlo) * D + u1) * D + u2) * ES : kOut;
  }
  const int csub = P::TP == 256 ? 0 : __builtin_amdgcn_readfirstlane(tid / P::TP);
  const In* in0 = static_cast<const In*>(a.in) + (int64_t)b * a.Cin * Ni + (int64_t)zlo * D * D;
  const int64_t nin = Ni - (int64_t)zlo * D * D;
  const int v = wave * 32 + li;
  const int lx = v % BoxT::BX, ly = (v / BoxT::BX) % BoxT::BY, lz = v / (BoxT::BX * BoxT::BY);
  const unsigned lbase = (unsigned)((lz * S * P::PY + ly * S) * P::PX + lx * S);
  const int K = a.Cin * K3, nch = (K + 15) / 16;
  const unsigned short* ap = a.ap + ((int64_t)blockIdx.y * MT * nch * 64 + lane) * 8;
  f32x16 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
  for (int c0 = 0; c0 < a.Cin; c0 += CG) {
    const int left = a.Cin - c0, nc = left < CG ? left : CG;
    const int chunks = left < CG ? (nc * K3 + 15) / 16 : KG / 16;
    const int nz = left < CG ? (chunks * 16 + K3 - 1) / K3 : CG;  // channels the k-steps reach
    if (c0) __syncthreads();  // the previous group's gathers are done
    // weights of the first PD chunks (the buffer ends a whole fragment row past the last one)
    const unsigned short* ag = ap + (int64_t)(c0 / CG) * (KG / 16) * 512;
    auto load_a = [&](int q, bf16x8 (&d)[MT]) {
      const int qq = q < chunks ? q : chunks - 1;
#pragma unroll
      for (int m = 0; m < MT; ++m) d[m] = *reinterpret_cast<const bf16x8*>(ag + ((int64_t)m * nch + qq) * 512);
    };
    bf16x8 av[PD][MT];
#pragma unroll
    for (int i = 0; i < PD; ++i) load_a(i, av[i]);
    // 16 channels of a position per batch, all requested before the first is converted and stored (the
    // scheduler would otherwise pair each load with its store).  Channels past the last one (they meet zero
    // weights) are stored as zero.
    constexpr int CSTEP = 256 / P::TP, CB = 16;
#pragma unroll
    for (int i = 0; i < P::NPOS; ++i) {
      const int e = tid % P::TP + P::TP * i;
#pragma unroll
      for (int cc = 0; cc < CG / CSTEP; cc += CB) {
        if (csub + CSTEP * cc >= nz) break;
        In h[CB];
#pragma unroll
        for (int k = 0; k < CB; ++k) {
          const int c = csub + CSTEP * (cc + k);
          const Rsrc r = rsrc(in0 + (int64_t)(c0 + (c < nc ? c : 0)) * Ni, nin);
          const unsigned off = c < nc ? pos[i] : kOut;
          if constexpr (BWD) h[k] = bload_h(r, off);
          else h[k] = bload_f(r, off);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (e < P::PV) {
#pragma unroll
          for (int k = 0; k < CB; ++k) {
            unsigned short v;
            if constexpr (BWD) v = h[k];
            else v = bf16_rn(h[k]);
            patch[(csub + CSTEP * (cc + k)) * P::PV + e] = v;
          }
        }
      }
    }
    __syncthreads();
    // chunk q: its weights were requested PD chunks ago, its operands one chunk ago, their offsets two
    auto load_t = [&](int q, uint4 (&f)[2]) {
      const int qq = q < chunks ? q : chunks - 1;
      f[0] = *reinterpret_cast<const uint4*>(&tab[qq * 16 + kh * 8]);
      f[1] = *reinterpret_cast<const uint4*>(&tab[qq * 16 + kh * 8 + 4]);
    };
    auto gather = [&](const uint4 (&f)[2]) {
      u16x8 h;
      h[0] = patch[lbase + f[0].x], h[1] = patch[lbase + f[0].y], h[2] = patch[lbase + f[0].z];
      h[3] = patch[lbase + f[0].w], h[4] = patch[lbase + f[1].x], h[5] = patch[lbase + f[1].y];
      h[6] = patch[lbase + f[1].z], h[7] = patch[lbase + f[1].w];
      return __builtin_bit_cast(bf16x8, h);
    };
    uint4 f[2];
    load_t(0, f);
    bf16x8 bv = gather(f);
    load_t(1, f);
    auto mult = [&](const bf16x8 (&w)[MT], const bf16x8& x) {
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[m], x, acc[m], 0, 0, 0);
    };
    int q0 = 0;
    for (; q0 + PD <= chunks; q0 += PD) {
#pragma unroll
      for (int i = 0; i < PD; ++i) {
        const bf16x8 cur = bv;
        bv = gather(f);
        load_t(q0 + i + 2, f);
        mult(av[i], cur);
        load_a(q0 + i + PD, av[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < PD - 1; ++i) {  // what a partial group leaves
      if (q0 + i >= chunks) break;
      const bf16x8 cur = bv;
      bv = gather(f);
      load_t(q0 + i + 2, f);
      mult(av[i], cur);
    }
  }
  const int z = o0[0] + lz, y = o0[1] + ly, x = o0[2] + lx;
  if (z >= Do || y >= Do || x >= Do) return;
  const int64_t o = ((int64_t)z * Do + y) * Do + x;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int c = m0 + m * 32 + acc_row(r, lane);
      if (c < a.M) {
        float w = acc[m][r];
        if (!BWD) {
          w += a.b[c];
          if (a.relu) w = w > 0.f ? w : 0.f;
        }
        a.y[((int64_t)b * a.M + c) * No + o] = w;
      }
    }
}

// Weights of every layer in fragment order, one launch (blockIdx.y: the layer):
// ap[tile][chunk][lane][j] = bf16 of A[tile 32 + lane % 32][chunk 16 + 8 (lane / 32) + j], A[co][ci k^3 + t] = W
// (forward) or A[ci][co k^3 + t] = W[co][ci][t] (data gradient); zero past the edges
struct PackArgs {
  struct Layer {
    const float* w;
    unsigned short* ap;
    int Cout, Cin, k3;
  } l[kMaxConvLayers];
};
__global__ __launch_bounds__(256) void k_pack_weights(PackArgs a, int bwd) {
  const PackArgs::Layer& L = a.l[blockIdx.y];
  const int Cin = L.Cin, k3 = L.k3;
  const int M = bwd ? Cin : L.Cout, K = (bwd ? L.Cout : Cin) * k3, nch = (K + 15) / 16;
  const int64_t n = (int64_t)((M + 31) / 32) * nch * 512;
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
    const int j = (int)(e & 7), lane = (int)(e >> 3) & 63;
    const int64_t r = e >> 9;
    const int q = (int)(r % nch), m = (int)(r / nch) * 32 + (lane & 31), k = q * 16 + 8 * (lane >> 5) + j;
    float v = 0.f;
    if (m < M && k < K) v = bwd ? L.w[((int64_t)(k / k3) * Cin + m) * k3 + k % k3] : L.w[(int64_t)m * K + k];
    L.ap[e] = bf16_rn(v);
  }
}

// Weight gradient: M = Cout, N = Cin k^3 (32 columns (ci, t) per wave), K = the voxels.  A workgroup walks
// boxes of 128 output voxels (box index blockIdx.z, blockIdx.z + gridDim.z, ...): it stages the box's G
// for its MT channel tiles and the input patch of the few channels its 128 columns touch as bf16 in LDS;
// a k-step is then 16 voxels, the A fragments 16-byte reads of G rows, the B fragment eight reads at
// constant offsets.  Its sums go to part[blockIdx.z] and are added up in a fixed order by k_sum_parts
// (the atomics that were here took a store of the whole gradient per 512 voxels).  The same batch: 2.17 ms
// -> 0.18 ms, and 0.07 ms for the sums.
struct WGradArgs {
  const float* x;           // [B][Cin][Di^3]
  const unsigned short* g;  // [B][Cout][Do^3] (bf16)
  float* part;              // [gridDim.z][Cout][Cin k^3]
  int B, Cin, Cout, Di, Do, pad, nb;
};
// RAGGED: some boxes reach past the output.  Their voxels there meet a G of zero, and an input that is not finite is
// kept from them (64^3 pairs have no such boxes: the test would cost a training step on 16 of them 11 of 1234 us).
template <class BoxT, int KS, int S, int MT, bool RAGGED>
__global__ __launch_bounds__(256) void k_conv_wgrad(WGradArgs a) {
  using P = Patch<BoxT, KS, S>;
  constexpr int K3 = KS * KS * KS;
  constexpr int XC = KS == 3 ? 6 : 128;  // channels that 128 columns touch at most
  constexpr int GL = 136;                // row stride of the staged G (16-byte rows, banks shifted by row)
  __shared__ unsigned short xs[XC * P::PV];
  __shared__ __align__(16) unsigned short gs[MT * 32 * GL];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 31, kh = lane >> 5;
  const int D = a.Di, Do = a.Do, N = a.Cin * K3;
  const int Ni = D * D * D, No = Do * Do * Do;
  const int n0 = blockIdx.x * 128, m0 = blockIdx.y * 32 * MT;
  const int cf = n0 / K3;  // first channel of the block's columns
  const int nlast = (n0 + 127 < N ? n0 + 127 : N - 1);
  const int nc = nlast / K3 - cf + 1;
  const int n = n0 + wave * 32 + li;
  const bool mine = n0 + wave * 32 < N;  // waves past the last column only stage
  const int nn = n < N ? n : N - 1;
  const int ci = nn / K3, t = nn - ci * K3, tz = t / (KS * KS), ty = (t / KS) % KS, tx = t % KS;
  const int xbase = (ci - cf) * P::PV + (tz * P::PY + ty) * P::PX + tx;
  f32x16 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
  const bool pairs = (Do & 1) == 0;  // two neighbours of a row in one load
  // the next box's operands are requested into registers before the current one is contracted
  constexpr int CSTEP = 256 / P::TP, XR = (XC + CSTEP - 1) / CSTEP, GR = MT * 8;
  const int csub = P::TP == 256 ? 0 : __builtin_amdgcn_readfirstlane(tid / P::TP);
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  float xr[P::NPOS][XR];
  unsigned gr[GR];
  const int gv = 2 * lane;  // G: two voxels of channel wave, wave + 4, ...
  const int gx = gv % BoxT::BX, gy = (gv / BoxT::BX) % BoxT::BY, gz = gv / (BoxT::BX * BoxT::BY);
  auto fetch = [&](int box) {
    const int b = box / a.nb;
    int o0[3];
    box_origin<BoxT>(box - b * a.nb, Do, o0);
    const int z0 = o0[0] * S - a.pad, zlo = z0 < 0 ? 0 : z0;
    unsigned pos[P::NPOS];
#pragma unroll
    for (int i = 0; i < P::NPOS; ++i) {
      const int e = tid % P::TP + P::TP * i;
      const int x = e % P::PX, y = (e / P::PX) % P::PY, z = e / (P::PX * P::PY);
      const int u0 = z0 + z, u1 = o0[1] * S + y - a.pad, u2 = o0[2] * S + x - a.pad;
      const bool ok = e < P::PV && u0 >= 0 && u1 >= 0 && u2 >= 0 && u0 < D && u1 < D && u2 < D;
      pos[i] = ok ? (unsigned)(((u0 - zlo) * D + u1) * D + u2) * 4u : kOut;
    }
    const float* xb = a.x + ((int64_t)b * a.Cin + cf) * Ni + (int64_t)zlo * D * D;
#pragma unroll
    for (int k = 0; k < XR; ++k) {
      const int c = csub + CSTEP * k;
      const Rsrc r = rsrc(xb + (int64_t)(c < nc ? c : 0) * Ni, (int64_t)Ni - (int64_t)zlo * D * D);
#pragma unroll
      for (int i = 0; i < P::NPOS; ++i) xr[i][k] = bload_f(r, c < nc ? pos[i] : kOut);
    }
    const int z = o0[0] + gz, y = o0[1] + gy, x = o0[2] + gx;
    const bool row = z < Do && y < Do, ok0 = row && x < Do, ok1 = row && x + 1 < Do;
    const unsigned go0 = ok0 ? (unsigned)((gz * Do + y) * Do + x) * 2u : kOut, go1 = ok1 ? go0 + 2u : kOut;
    const unsigned short* gb = a.g + (int64_t)b * a.Cout * No + (int64_t)o0[0] * Do * Do;
#pragma unroll
    for (int k = 0; k < GR; ++k) {
      const int c = m0 + uwave + 4 * k;
      const bool in = c < a.Cout;
      const Rsrc r = rsrc(gb + (int64_t)(in ? c : 0) * No, (int64_t)No - (int64_t)o0[0] * Do * Do);
      // x and the rows even: both voxels lie in the row, 4-byte aligned
      if (pairs) gr[k] = (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)(in ? go0 : kOut), 0, 0);
      else gr[k] = bload_h(r, in ? go0 : kOut) | ((unsigned)bload_h(r, in ? go1 : kOut) << 16);
    }
  };
  const int total = a.nb * a.B;
  int box = blockIdx.z;
  if (box < total) fetch(box);
  for (; box < total; box += gridDim.z) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < P::NPOS; ++i) {
      const int e = tid % P::TP + P::TP * i;
      if (e < P::PV) {
#pragma unroll
        for (int k = 0; k < XR; ++k) {
          const int c = csub + CSTEP * k;
          if (c < XC) xs[c * P::PV + e] = bf16_rn(xr[i][k]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < GR; ++k) *reinterpret_cast<unsigned*>(&gs[(wave + 4 * k) * GL + gv]) = gr[k];
    __syncthreads();
    if (box + (int)gridDim.z < total) fetch(box + gridDim.z);
    if (mine) {
      int o0[3];
      if constexpr (RAGGED) box_origin<BoxT>(box % a.nb, Do, o0);
#pragma unroll
      for (int q = 0; q < 8; ++q) {  // voxels 16 q + 8 kh + j: eight neighbours of one box row
        const int v = 16 * q + 8 * kh;
        const int lx = v % BoxT::BX, ly = (v / BoxT::BX) % BoxT::BY, lz = v / (BoxT::BX * BoxT::BY);
        const unsigned short* xp = xs + xbase + (lz * S * P::PY + ly * S) * P::PX + lx * S;
        u16x8 h;
#pragma unroll
        for (int j = 0; j < 8; ++j) h[j] = xp[j * S];
        if constexpr (RAGGED) {
          const int left = o0[0] + lz < Do && o0[1] + ly < Do ? Do - o0[2] - lx : 0;
#pragma unroll
          for (int j = 0; j < 8; ++j) h[j] = j < left ? h[j] : (unsigned short)0;
        }
        const bf16x8 bv = __builtin_bit_cast(bf16x8, h);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const bf16x8 av = *reinterpret_cast<const bf16x8*>(&gs[(m * 32 + li) * GL + v]);
          acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[m], 0, 0, 0);
        }
      }
    }
  }
  if (n < N) {
    float* out = a.part + (int64_t)blockIdx.z * a.Cout * N;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = m0 + m * 32 + acc_row(r, lane);
        if (c < a.Cout) out[(int64_t)c * N + n] = acc[m][r];
      }
  }
}

// dw[i] += sum_z part[z][i]
// (G waves share out the parts of 64 weights: a small layer has many parts and few weights, whose one thread each
// then read 512 parts in turn, 23.5 -> 4.3 us)
template <int G>
__global__ __launch_bounds__(64 * G) void k_sum_parts(float* __restrict__ dw, const float* __restrict__ part, int64_t n,
                                                      int z) {
  __shared__ float sums[G][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = blockIdx.x * (int64_t)64 + lane;
  const int per = (z + G - 1) / G, k1 = min(z, (wave + 1) * per);
  float s = 0.f;
  if (i < n) {
#pragma unroll 8
    for (int k = wave * per; k < k1; ++k) s += part[(int64_t)k * n + i];
  }
  sums[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < n) {
#pragma unroll
    for (int g = 1; g < G; ++g) s += sums[g][lane];
    dw[i] += s;
  }
}

// G = dY * act'(Y) as the bf16 operand of both gradients, and the bias gradient db[c] += sum over the
// block's slice of G[b][c][:] (8192 voxels per block: one atomic per slice instead of one per 256 voxels)
constexpr int kActSlice = 8192;
__global__ __launch_bounds__(256) void k_act_bwd(const float* __restrict__ dy, const float* __restrict__ y,
                                                 unsigned short* __restrict__ g, float* db, int C, int No, int relu) {
  const int bc = blockIdx.y;  // b * C + c
  const int c = bc % C;
  const int lo = blockIdx.x * kActSlice, hi = min(No, lo + kActSlice);
  const int64_t base = (int64_t)bc * No;
  float s = 0.f;
#pragma unroll 4
  for (int o = lo + threadIdx.x; o < hi; o += 256) {
    float v = dy[base + o];
    if (relu && y[base + o] <= 0.f) v = 0.f;
    g[base + o] = bf16_rn(v);
    s += v;
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  __shared__ float part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(&db[c], part[0] + part[1] + part[2] + part[3]);
}

__global__ void k_adam(float* w, float* m, float* v, const float* g, int64_t n, float lr, float b1, float b2,
                       float c1, float c2, float eps) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void k_fill(float* p, int64_t n, float v) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// network input from an image pair: box average of each f0 x f1 x f2 voxel cell, out [2][S^3].  F > 0: cells of F^3,
// whose loads are then all requested before the first sum (the loops of any other cell wait for a load per row:
// 128^3 to 64^3 8.5 -> 5.7 us, 16.8 MB)
template <int F>
__global__ __launch_bounds__(256) void k_pool_pair(const float* __restrict__ I0, const float* __restrict__ I1, int n1,
                                                   int n2, int f0, int f1, int f2, int S, float* __restrict__ out) {
  const int64_t S3 = (int64_t)S * S * S;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= 2 * S3) return;
  if constexpr (F > 0) f0 = f1 = f2 = F;
  const int ch = e >= S3;
  const unsigned o = (unsigned)(e - ch * S3), q = o / (unsigned)S;
  const int oz = (int)(q / (unsigned)S), oy = (int)(q % (unsigned)S), ox = (int)(o % (unsigned)S);
  const float* __restrict__ I = ch == 0 ? I0 : I1;
  auto row = [&](int a, int b) { return I + ((int64_t)(oz * f0 + a) * n1 + (oy * f1 + b)) * n2 + (int64_t)ox * f2; };
  float sum = 0.f;
  if constexpr (F > 0) {
    float v[F][F][F];
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b)
#pragma unroll
        for (int c = 0; c < F; ++c) v[a][b][c] = row(a, b)[c];
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b)
#pragma unroll
        for (int c = 0; c < F; ++c) sum += v[a][b][c];
  } else {
    for (int a = 0; a < f0; ++a)
      for (int b = 0; b < f1; ++b)
        for (int c = 0; c < f2; ++c) sum += row(a, b)[c];
  }
  out[e] = sum / (float)(f0 * f1 * f2);
}

// Coarse velocity samples [B][3][s^3] <-> band-limited coefficients [B][3][K0][K1][K2], one axis per launch:
// the separable projection P[a][x] onto the s-point band for slots a < s - 1 (zero elsewhere), and its
// transpose for the loss gradient.  Each thread forms one value of a stage as a sum of at most s terms, in the
// order of the nested sum over (x0, x1, x2) whose inner sums every output of that line shares (16^3 samples:
// 48 terms per output instead of 16^3; 522 -> 11 us for one pair's velocity, 3.9 ms -> 13 us for a batch of 16).

// t[bc][row][a] = sum_x P[a][x] in[bc][row][x] over the innermost axis (a < nb); rows of a channel: s^2
__global__ __launch_bounds__(256) void k_samples_axis2(const float* __restrict__ samp, const float* __restrict__ P,
                                                       int64_t total, int gs, int sz, float* __restrict__ t) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  const int nb = sz - 1, s2 = sz * sz;
  const int a2 = (int)(e % nb);
  const int64_t r = e / nb, bc = r / s2;
  const int row = (int)(r - bc * s2);
  const int64_t sc = (bc / 3) * gs * 3 + bc % 3;  // sample channel: group b at stride gs
  const float* sp = samp + (sc * s2 + row) * sz;
  float v = 0.f;
#pragma unroll 4
  for (int x2 = 0; x2 < sz; ++x2) v += P[a2 * sz + x2] * sp[x2];
  t[e] = v;
}
// u[bc][x0][a1][a2] = sum_x1 P[a1][x1] t[bc][x0][x1][a2]
__global__ __launch_bounds__(256) void k_samples_axis1(const float* __restrict__ t, const float* __restrict__ P,
                                                       int64_t total, int sz, float* __restrict__ u) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  const int nb = sz - 1;
  const int a2 = (int)(e % nb), a1 = (int)((e / nb) % nb);
  const float* tp = t + (e / ((int64_t)nb * nb)) * sz * nb + a2;
  float v = 0.f;
#pragma unroll 4
  for (int x1 = 0; x1 < sz; ++x1) v += P[a1 * sz + x1] * tp[x1 * nb];
  u[e] = v;
}
// v[bc][a0][a1][a2] = sum_x0 P[a0][x0] u[bc][x0][a1][a2] inside the block, 0 in every other slot
__global__ __launch_bounds__(256) void k_samples_axis0(const float* __restrict__ u, const float* __restrict__ P,
                                                       int64_t total, int sz, int k0, int k1, int k2,
                                                       float* __restrict__ v) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  const int64_t Q = (int64_t)k0 * k1 * k2, bc = e / Q, q = e - bc * Q;
  const int a0 = (int)(q / ((int64_t)k1 * k2)), a1 = (int)((q / k2) % k1), a2 = (int)(q % k2);
  const int nb = sz - 1;
  float r = 0.f;
  if (a0 < nb && a1 < nb && a2 < nb) {
    const float* up = u + bc * sz * nb * nb + a1 * nb + a2;
#pragma unroll 4
    for (int x0 = 0; x0 < sz; ++x0) r += P[a0 * sz + x0] * up[(int64_t)x0 * nb * nb];
  }
  v[e] = r;
}

// gradient of the weighted squared coefficient error with respect to the samples, the same stages transposed:
// ds[b][c][x] = scale * sum_{a in block} P[a0][x0] P[a1][x1] P[a2][x2] w[a] diff[b][c][a]
__global__ __launch_bounds__(256) void k_block_axis2(const float* __restrict__ diff, const double* __restrict__ w,
                                                     const float* __restrict__ P, int64_t total, int sz, int k0, int k1,
                                                     int k2, float* __restrict__ t) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  const int nb = sz - 1;
  const int x2 = (int)(e % sz), a1 = (int)((e / sz) % nb), a0 = (int)((e / ((int64_t)sz * nb)) % nb);
  const int64_t bc = e / ((int64_t)sz * nb * nb), q0 = ((int64_t)a0 * k1 + a1) * k2;
  const float* dp = diff + bc * k0 * k1 * k2 + q0;
  float v = 0.f;
#pragma unroll 4
  for (int a2 = 0; a2 < nb; ++a2) v += P[a2 * sz + x2] * (float)w[q0 + a2] * dp[a2];
  t[e] = v;
}
__global__ __launch_bounds__(256) void k_block_axis1(const float* __restrict__ t, const float* __restrict__ P,
                                                     int64_t total, int sz, float* __restrict__ u) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  const int nb = sz - 1;
  const int x2 = (int)(e % sz), x1 = (int)((e / sz) % sz);
  const float* tp = t + (e / ((int64_t)sz * sz)) * nb * sz + x2;
  float v = 0.f;
#pragma unroll 4
  for (int a1 = 0; a1 < nb; ++a1) v += P[a1 * sz + x1] * tp[a1 * sz];
  u[e] = v;
}
__global__ __launch_bounds__(256) void k_block_axis0(const float* __restrict__ u, const float* __restrict__ P,
                                                     int64_t total, int gs, int sz, float scale,
                                                     float* __restrict__ ds) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e >= total) return;
  const int nb = sz - 1, s2 = sz * sz;
  const int64_t s3 = (int64_t)s2 * sz, bc = e / s3;
  const int x = (int)(e - bc * s3), x0 = x / s2, x12 = x - x0 * s2;
  const int64_t sc = (bc / 3) * gs * 3 + bc % 3;  // output channel: group b at stride gs
  const float* up = u + bc * nb * s2 + x12;
  float r = 0.f;
#pragma unroll 4
  for (int a0 = 0; a0 < nb; ++a0) r += P[a0 * sz + x0] * up[(int64_t)a0 * s2];
  ds[sc * s3 + x] = scale * r;
}

}  // namespace

// ------------------------------------------------------------------------------------------
namespace {

// picks the box of an output edge: the widest whose rows are full
template <class F>
void with_box(int Do, F&& f) {
  if (Do >= 24) f(BoxWide{});
  else if (Do > 8) f(BoxMid{});
  else f(BoxSmall{});
}
template <class BoxT>
int boxes(int Do) {
  return ceil_div(Do, BoxT::BX) * ceil_div(Do, BoxT::BY) * ceil_div(Do, BoxT::BZ);
}

// MT channel tiles per workgroup share a gathered operand; fewer when that would leave CUs without a
// workgroup (two per CU wanted)
template <class BoxT, int KS, int S, bool BWD>
void launch_conv(const char* name, double bytes, double flops, ConvArgs a, int B, hipStream_t s) {
  a.nb = boxes<BoxT>(a.Do);
  const int tiles = ceil_div(a.M, 32);
  int mt = tiles >= 3 ? 4 : tiles;
  while (mt > 1 && (int64_t)a.nb * B * ceil_div(tiles, mt) < 512) mt >>= 1;
  dim3 g(a.nb, ceil_div(tiles, mt), B);
  if (mt == 1) prof::launch(name, bytes, flops, k_conv<BoxT, KS, S, 1, BWD>, g, dim3(256), 0, s, a);
  else if (mt == 2) prof::launch(name, bytes, flops, k_conv<BoxT, KS, S, 2, BWD>, g, dim3(256), 0, s, a);
  else prof::launch(name, bytes, flops, k_conv<BoxT, KS, S, 4, BWD>, g, dim3(256), 0, s, a);
  LDDMM_LAUNCH_CHECK();
}

template <class BoxT, int KS, int S, bool RAGGED>
void launch_wgrad(double flops, const WGradArgs& a, int mt, dim3 g, hipStream_t s) {
  const char* name = "k_conv_bwd_weight";
  auto go = [&](auto* k) { prof::launch(name, 0.0, flops, k, g, dim3(256), 0, s, a); };
  if (mt == 1) go(k_conv_wgrad<BoxT, KS, S, 1, RAGGED>);
  else if (mt == 2) go(k_conv_wgrad<BoxT, KS, S, 2, RAGGED>);
  else if constexpr (KS == 3) go(k_conv_wgrad<BoxT, KS, S, 4, RAGGED>);
  LDDMM_LAUNCH_CHECK();
}
template <class BoxT, int KS, int S>
void launch_wgrad(double flops, const WGradArgs& a, int mt, dim3 g, hipStream_t s) {
  if (a.Do % BoxT::BX || a.Do % BoxT::BY || a.Do % BoxT::BZ) launch_wgrad<BoxT, KS, S, true>(flops, a, mt, g, s);
  else launch_wgrad<BoxT, KS, S, false>(flops, a, mt, g, s);
}

int out_edge(const ConvLayer& L, int Di) { return (Di + 2 * L.pad - L.k) / L.stride + 1; }

void check_layer(const ConvLayer& L, int Di, int B) {
  if (!((L.k == 3 && (L.stride == 1 || L.stride == 2)) || (L.k == 1 && L.stride == 1)) || L.pad < 0 || L.pad >= L.k)
    throw ArgError("convolution: kernels of 3^3 with stride 1 or 2, or 1^3 with stride 1");
  if (B < 1 || Di < 1 || (int64_t)Di * Di * Di >= (int64_t(1) << 31)) throw ArgError("convolution: size");
}

}  // namespace

int64_t packed_elems(const ConvLayer& L) {
  const int64_t k3 = (int64_t)L.k * L.k * L.k;
  const int64_t f = (int64_t)ceil_div(L.cout, 32) * ceil_div(L.cin * k3, 16), b = (int64_t)ceil_div(L.cin, 32) * ceil_div(L.cout * k3, 16);
  // a workgroup of 2 or 4 channel tiles reads whole groups of tiles
  return 512 * (std::max(f, b) + 3 * ceil_div(std::max(L.cin, L.cout) * k3, 16));
}

// Voxel splits of a layer's weight gradient: about two workgroups per CU, bounded by the boxes and by the
// partial gradients' memory (64 MB)
static int wgrad_mt(const ConvLayer& L) {
  const int t = ceil_div(L.cout, 32);
  return t >= 3 && L.k == 3 ? 4 : t >= 2 ? 2 : 1;
}
static int wgrad_splits(const ConvLayer& L, int B, int Do) {
  int nb = 0;
  with_box(Do, [&](auto bx) { nb = boxes<decltype(bx)>(Do); });
  const int64_t per = (int64_t)ceil_div(L.cin * L.k * L.k * L.k, 128) * ceil_div(ceil_div(L.cout, 32), wgrad_mt(L));
  int64_t z = std::max<int64_t>(1, 512 / per);
  z = std::min<int64_t>(z, (int64_t)nb * B);
  return (int)std::max<int64_t>(1, std::min<int64_t>(z, (int64_t(1) << 24) / L.nw()));
}
int64_t wgrad_part_elems(const ConvLayer& L, int B, int Di) {
  return wgrad_splits(L, B, out_edge(L, Di)) * L.nw();
}

void pack_weights(const ConvLayer* L, unsigned short* const* ap, int n, bool bwd, hipStream_t s) {
  if (n < 1) return;
  if (n > kMaxConvLayers) throw ArgError("too many convolution layers");
  PackArgs a{};
  int64_t most = 0;
  for (int i = 0; i < n; ++i) {
    const int k3 = L[i].k * L[i].k * L[i].k, M = bwd ? L[i].cin : L[i].cout, K = (bwd ? L[i].cout : L[i].cin) * k3;
    a.l[i] = {L[i].w, ap[i], L[i].cout, L[i].cin, k3};
    most = std::max(most, (int64_t)ceil_div(M, 32) * ceil_div(K, 16) * 512);
  }
  k_pack_weights<<<dim3(std::min(1024, ceil_div(most, 256)), n), 256, 0, s>>>(a, bwd ? 1 : 0);
  LDDMM_LAUNCH_CHECK();
}

void conv_forward(const ConvLayer& L, const float* x, float* y, int B, int Di, const unsigned short* packed, hipStream_t s) {
  check_layer(L, Di, B);
  ConvArgs a{};
  a.in = x, a.ap = packed, a.b = L.b, a.y = y;
  a.Cin = L.cin, a.M = L.cout, a.pad = L.pad, a.up = 1, a.relu = L.relu;
  a.Di = Di, a.Do = out_edge(L, Di);
  const double No = (double)a.Do * a.Do * a.Do, Ni = (double)Di * Di * Di;
  const double bytes = 4.0 * (B * L.cin * Ni + B * L.cout * No), flops = 2.0 * B * No * L.cout * L.cin * L.k * L.k * L.k;
  with_box(a.Do, [&](auto bx) {
    using BoxT = decltype(bx);
    if (L.k == 1) launch_conv<BoxT, 1, 1, false>("k_conv_fwd", bytes, flops, a, B, s);
    else if (L.stride == 1) launch_conv<BoxT, 3, 1, false>("k_conv_fwd", bytes, flops, a, B, s);
    else launch_conv<BoxT, 3, 2, false>("k_conv_fwd", bytes, flops, a, B, s);
  });
}

void conv_backward(const ConvLayer& L, const float* x, const float* y, const float* dy, unsigned short* g, float* dx,
                   int B, int Di, const unsigned short* packed, float* part, hipStream_t s) {
  check_layer(L, Di, B);
  const int Do = out_edge(L, Di), No = Do * Do * Do, k3 = L.k * L.k * L.k;
  // activation derivative and bias gradient
  dim3 ga(ceil_div(No, kActSlice), B * L.cout);
  k_act_bwd<<<ga, 256, 0, s>>>(dy, y, g, L.db, L.cout, No, L.relu);
  LDDMM_LAUNCH_CHECK();
  // weight gradient (accumulated)
  WGradArgs w{};
  w.x = x, w.g = g, w.part = part;
  w.B = B, w.Cin = L.cin, w.Cout = L.cout, w.Di = Di, w.Do = Do, w.pad = L.pad;
  const int N = L.cin * k3, mt = wgrad_mt(L), z = wgrad_splits(L, B, Do);
  with_box(Do, [&](auto bx) {
    using BoxT = decltype(bx);
    w.nb = boxes<BoxT>(Do);
    dim3 gw(ceil_div(N, 128), ceil_div(ceil_div(L.cout, 32), mt), z);
    const double flops = 2.0 * B * (double)No * L.cout * N;
    if (L.k == 1) launch_wgrad<BoxT, 1, 1>(flops, w, mt, gw, s);
    else if (L.stride == 1) launch_wgrad<BoxT, 3, 1>(flops, w, mt, gw, s);
    else launch_wgrad<BoxT, 3, 2>(flops, w, mt, gw, s);
  });
  if (z >= 128) k_sum_parts<16><<<ceil_div(L.nw(), 64), 1024, 0, s>>>(L.dw, part, L.nw(), z);
  else k_sum_parts<4><<<ceil_div(L.nw(), 64), 256, 0, s>>>(L.dw, part, L.nw(), z);
  LDDMM_LAUNCH_CHECK();
  if (dx) {
    ConvArgs a{};
    a.in = g, a.ap = packed, a.y = dx;
    a.Cin = L.cout, a.M = L.cin, a.pad = L.pad, a.up = L.stride, a.relu = 0;
    a.Di = Do, a.Do = Di;
    const double flops = 2.0 * B * (double)Di * Di * Di * L.cin * L.cout * k3;
    with_box(Di, [&](auto bx) {
      using BoxT = decltype(bx);
      if (L.k == 1) launch_conv<BoxT, 1, 1, true>("k_conv_bwd_data", 0.0, flops, a, B, s);
      else launch_conv<BoxT, 3, 1, true>("k_conv_bwd_data", 0.0, flops, a, B, s);
    });
  }
}

void adam_step(float* w, float* m, float* v, const float* g, int64_t n, float lr, int t, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, (float)t), c2 = 1.f - std::pow(b2, (float)t);
  k_adam<<<ceil_div(n, 256), 256, 0, s>>>(w, m, v, g, n, lr, b1, b2, c1, c2, 1e-8f);
  LDDMM_LAUNCH_CHECK();
}

void fill(float* p, int64_t n, float v, hipStream_t s) {
  if (n <= 0) return;
  k_fill<<<ceil_div(n, 256), 256, 0, s>>>(p, n, v);
  LDDMM_LAUNCH_CHECK();
}

void pool_pair(const float* I0, const float* I1, const int n[3], int S, float* out, hipStream_t s) {
  const int64_t tot = 2LL * S * S * S;
  const int f0 = n[0] / S, f1 = n[1] / S, f2 = n[2] / S;
  auto* k = f0 == 2 && f1 == 2 && f2 == 2 ? k_pool_pair<2> : f0 == 1 && f1 == 1 && f2 == 1 ? k_pool_pair<1> : k_pool_pair<0>;
  k<<<ceil_div(tot, 256), 256, 0, s>>>(I0, I1, n[1], n[2], f0, f1, f2, S, out);
  LDDMM_LAUNCH_CHECK();
}

int64_t stage_elems(int B, int sz) { return 2LL * B * 3 * sz * sz * sz; }

void samples_to_bl(const float* samp, const float* P, int B, int gs, int sz, const int k[3], float* v, float* ws,
                   hipStream_t s) {
  const int64_t nb = sz - 1, bc = (int64_t)B * 3, n2 = bc * sz * sz * nb, n1 = bc * sz * nb * nb, n0 = bc * k[0] * k[1] * k[2];
  float* u = ws + bc * sz * sz * sz;
  if (nb > 0) {
    k_samples_axis2<<<ceil_div(n2, 256), 256, 0, s>>>(samp, P, n2, gs, sz, ws);
    k_samples_axis1<<<ceil_div(n1, 256), 256, 0, s>>>(ws, P, n1, sz, u);
  }
  k_samples_axis0<<<ceil_div(n0, 256), 256, 0, s>>>(u, P, n0, sz, k[0], k[1], k[2], v);
  LDDMM_LAUNCH_CHECK();
}

void block_grad(const float* diff, const double* w, const float* P, int B, int gs, int sz, const int k[3],
                float scale, float* ds, float* ws, hipStream_t s) {
  const int64_t nb = sz - 1, bc = (int64_t)B * 3, n2 = bc * nb * nb * sz, n1 = bc * nb * sz * sz, n0 = bc * sz * sz * sz;
  float* u = ws + bc * sz * sz * sz;
  if (nb > 0) {
    k_block_axis2<<<ceil_div(n2, 256), 256, 0, s>>>(diff, w, P, n2, sz, k[0], k[1], k[2], ws);
    k_block_axis1<<<ceil_div(n1, 256), 256, 0, s>>>(ws, P, n1, sz, u);
  }
  k_block_axis0<<<ceil_div(n0, 256), 256, 0, s>>>(u, P, n0, gs, sz, scale, ds);
  LDDMM_LAUNCH_CHECK();
}

}  // namespace lddmm
