// Internal interface of the proposal network's kernels (amh_nn.hip).
// Activations are NHWC bf16 with channel counts that are multiples of 16;
// weights are [cout_pad][kpad] with k = tap * cin + c, tap = ky * ks + kx,
// kpad = ks^2 cin rounded up to 32, padded entries zero.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

#include "amh_bf16.h"

namespace amh {
namespace nn {

constexpr int kHeadPitch = 8;   // floats per cell of the head's output (5 used)
constexpr int kMaxSplits = 64;  // pixel splits of a weight gradient
constexpr int kMaxLayers = 12;

// depth head: depth = 1 / clamp(q_ref + R tanh(z0), q_far, q_near)
struct DepthHead {
    float d_min, d_max, q_far, q_near, R;
};

struct Conv3Args {
    const bf16_t *x;             // [n*h*w][cin - c1]
    const bf16_t *low = nullptr;  // concatenation: [n*h/2*w/2][c1] upsampled before x's channels
    const bf16_t *wgt;           // [cout][kpad]
    const float *bias = nullptr;  // [cout]
    const bf16_t *mask = nullptr;  // [n*h*w][cout]: outputs where mask <= 0 are zeroed
    bf16_t *y;                   // [n*h*w][cout]
    bf16_t *pool = nullptr;      // [n*h/2*w/2][cout]: 2 x 2 means of y
    bf16_t *xcopy = nullptr;     // kept copy of x
    int n, h, w;
    int relu = 0;
    int tiles_x = 0, tiles_y = 0;  // set by the launch
    // the 1x1 head on y (16 channels)
    const bf16_t *head_w = nullptr;  // [16][32]
    const float *head_b = nullptr;   // [16]
    const float *q_ref = nullptr;    // [n*h*w], copied to q_copy
    float *q_copy = nullptr, *z = nullptr;  // z [n*h*w][kHeadPitch]
    float *out = nullptr;        // [n*h*w][5] or NULL
    DepthHead dh = {};
};

struct WgradArgs {
    const bf16_t *x;       // [n*h*w][cin - c1] layer input
    const bf16_t *low;     // its first c1 channels at half the resolution (concatenation), c1 = 0 otherwise
    const bf16_t *g;       // [n*h*w][cout_pad] gradient at the layer's pre-activation
    float *part;           // [splits][cout_pad][kpad]
    float *bpart;          // [splits][cout_pad]
    int n, h, w;
    int cin, c1, cout_pad, kpad, ks;
    int chunk;             // pixels per split (multiple of 32)
};

// where a layer's parameters lie in the padded arrays (weights at w_off, biases at b_off), its transposed weights at
// t_off; partial sums at kMaxSplits times those offsets
struct LayerDims {
    int cin, cout_pad, kpad, kpad_t, taps;
    int w_off, b_off, t_off;
    int splits;
};
struct LayerTable {
    int n;
    LayerDims l[kMaxLayers];
};

hipError_t launch_conv3(int cin, int cout, const Conv3Args &a, hipStream_t s);
hipError_t launch_head_grad(const bf16_t *g, const bf16_t *wgt, const bf16_t *mask, int P, bf16_t *out, hipStream_t s);
hipError_t launch_wgrad(const WgradArgs &a, int splits, hipStream_t s);
hipError_t launch_wgrad_reduce(const LayerTable &tab, const float *part, int n_pad, float *grad, hipStream_t s);
hipError_t launch_transpose_w(const LayerTable &tab, const bf16_t *w, int n, bf16_t *wt, hipStream_t s);
hipError_t launch_enc_grad(const bf16_t *dp, const bf16_t *dcat, int Ccat, int off, const bf16_t *e_act, int n, int h,
                           int w, int C, bf16_t *g, hipStream_t s);
hipError_t launch_up_grad(const bf16_t *dcat, int Ccat, const bf16_t *act, int n, int h, int w, int C1, bf16_t *g,
                          hipStream_t s);
int loss_blocks(int P);
hipError_t launch_loss(const float *z, const float *q_ref, const float *target, int P, const DepthHead &dh, bf16_t *dz,
                       float *part, float *loss, hipStream_t s);
hipError_t launch_adam(float *p, const float *g, float *m, float *v, bf16_t *pb, int n, float lr, float b1, float b2,
                       float eps, int step, hipStream_t s);
hipError_t launch_to_bf16(const float *src, int n, bf16_t *dst, hipStream_t s);
hipError_t launch_targets(const float *depth, const float *normal, const float *cost, int W, int H, int cell,
                          int h4, int w4, float beta, float *target, hipStream_t s);

}  // namespace nn
}  // namespace amh
