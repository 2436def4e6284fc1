// Small 3D convolutional network of the learned warm start (see nn.hip).
#pragma once

#include "common.h"

namespace lddmm {

struct ConvLayer {
  int cin = 0, cout = 0, k = 3, stride = 1, pad = 1, relu = 1;
  float *w = nullptr, *b = nullptr;    // float masters [cout][cin][k^3], [cout]
  float *dw = nullptr, *db = nullptr;  // gradients
  float *mw = nullptr, *vw = nullptr, *mb = nullptr, *vb = nullptr;  // Adam moments
  int64_t nw() const { return (int64_t)cout * cin * k * k * k; }
};

// Weights in the convolution kernels' operand order (bf16): layer i's into ap[i], packed_elems(L[i]) values, for
// the forward pass or the data gradient.  Packed anew for every pass: the master weights may have changed.
constexpr int kMaxConvLayers = 8;
int64_t packed_elems(const ConvLayer& L);
void pack_weights(const ConvLayer* L, unsigned short* const* ap, int n, bool bwd, hipStream_t s);
// x, y float [B][channels][edge^3]; packed: the layer's packed weights
void conv_forward(const ConvLayer& L, const float* x, float* y, int B, int Di, const unsigned short* packed,
                  hipStream_t s);
// g: bf16 scratch of y's size; part: scratch of wgrad_part_elems floats; dx may be null (first layer)
int64_t wgrad_part_elems(const ConvLayer& L, int B, int Di);
void conv_backward(const ConvLayer& L, const float* x, const float* y, const float* dy, unsigned short* g, float* dx,
                   int B, int Di, const unsigned short* packed, float* part, hipStream_t s);
void adam_step(float* w, float* m, float* v, const float* g, int64_t n, float lr, int t, hipStream_t s);
void fill(float* p, int64_t n, float v, hipStream_t s);
// box-average an image pair of n[0] x n[1] x n[2] voxels (each divisible by S) into a [2][S^3] input
void pool_pair(const float* I0, const float* I1, const int n[3], int S, float* out, hipStream_t s);
// coarse samples -> band coefficients [B][3][k0][k1][k2] through the projection P [sz][sz]; group b
// of three sample channels starts at channel 3 gs b of samp ([B][3 gs][sz^3])
// (ws: scratch of stage_elems(B, sz) floats, in both maps)
int64_t stage_elems(int B, int sz);
void samples_to_bl(const float* samp, const float* P, int B, int gs, int sz, const int k[3], float* v, float* ws,
                   hipStream_t s);
// ds = scale * (projection block)^T (w * diff), diff [B][3][k0][k1][k2], w [k0 k1 k2] (double), written
// to the channels 3 gs b .. 3 gs b + 2 of ds ([B][3 gs][sz^3]); other channels are left untouched
void block_grad(const float* diff, const double* w, const float* P, int B, int gs, int sz, const int k[3],
                float scale, float* ds, float* ws, hipStream_t s);

}  // namespace lddmm
