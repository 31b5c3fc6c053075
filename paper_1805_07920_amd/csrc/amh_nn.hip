// gfx950 kernels of the proposal network: a 4-level convolutional
// encoder-decoder over bf16 NHWC activations with fp32 accumulation on the
// matrix cores, its backward pass, the training loss and Adam.
//
// Convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16:
//   forward / input gradient: rows = 16 output channels, columns = 16 pixels,
//     K = taps x input channels (padded to a multiple of 32 with zero weights);
//     each lane feeds 8 consecutive channels of one tap of one pixel, one
//     16-byte LDS read;
//   weight gradient: rows = 16 output channels, columns = 16 (tap, channel)
//     pairs, K = pixels, split over workgroups into partial sums that a second
//     kernel adds in a fixed order (deterministic, no atomics).
// The input gradient is a forward convolution of the output gradient with the
// weights transposed and the taps mirrored; the ReLU of the layer below is
// applied in its epilogue as a mask.  All channel counts are multiples of 16.
#include <hip/hip_runtime.h>

#include "amh_bf16.h"
#include "amh_nn.h"

namespace amh {
namespace nn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define NN_LAUNCH(...)                   \
    do {                                 \
        (void)hipGetLastError();         \
        hipLaunchKernelGGL(__VA_ARGS__); \
    } while (0)

__device__ __forceinline__ float sigmoidf(float z) { return 1.f / (1.f + __expf(-z)); }

// depth head: q = clamp(q_ref + R tanh(z0), q_far, q_near); returns q and dq/dz0 (0 where clamped)
__device__ __forceinline__ float head_q(float z0, float q_ref, const DepthHead &dh, float &dq) {
    const float th = tanhf(z0);
    const float u = fmaf(dh.R, th, q_ref);
    const bool inside = u > dh.q_far && u < dh.q_near;
    dq = inside ? dh.R * (1.f - th * th) : 0.f;
    return fminf(fmaxf(u, dh.q_far), dh.q_near);
}

// the value held by the other lane of the pair (lanes 2 i, 2 i + 1)
__device__ __forceinline__ float pair_swap(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
}

// ---------------------------------------------------------------------------
// 3x3 convolution (forward, and input gradient with transposed weights).
//
// A workgroup of 4 waves takes 16 x TH pixels of one image and every output
// channel: the input tile with its one-pixel halo is staged in LDS (zeros
// outside the image; a concatenation's two sources are read where they lie,
// the low-resolution one at half the coordinates), and the weights are the
// MFMA's first operand, read straight from the cache.  A lane then holds 4
// consecutive channels of one pixel: 8-byte stores, the pooled half-resolution
// map from the neighbouring lane and row, the head's product and decoding,
// all in the same launch.  Pixels of the LDS tile are 2 CIN + 16 bytes apart,
// an odd multiple of 16 bytes, so the 16 lanes of a row group read on
// disjoint banks.
//
// Bound: launches and the latency of one tile's load and K / 32 dependent
// MFMAs (8.3 GFLOP, 60 MB through the caches); the order of the sums over K is
// fixed (steps of 32 from tap 0), whatever the tile.  Forward at 320 x 480
// cells: 21 launches of kernels without LDS, scattered 2-byte stores and a
// division per step took 221 us; 85 us with 11.
// ---------------------------------------------------------------------------
constexpr int kTileX = 16;

// CIN input channels, the first C1 of them from the half-resolution source (0: one source); COUT output channels; WN
// of the 4 waves split the output channels, the others the rows, NG rows each; POOL: also the 2 x 2 means; HEAD: also
// the 1x1 head and its decoding
template <int CIN, int COUT, int C1, int WN, int NG, bool POOL, bool HEAD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HEAD ? 5 : 1))) void conv3_kernel(Conv3Args a) {
    constexpr int NT = COUT / 16, NTW = (NT + WN - 1) / WN, TH = 4 / WN * NG;
    constexpr int SW = kTileX + 2, SH = TH + 2, PXS = CIN * 2 + 16, C8 = CIN / 8;
    constexpr int K = 9 * CIN, STEPS = (K + 31) / 32, KPAD = STEPS * 32;
    static_assert(!POOL || NG == 2, "a wave pools its own two rows");
    static_assert(!HEAD || (COUT == 16 && WN == 1), "the head reads a pixel's 16 channels");
    __shared__ __align__(16) unsigned char tile[SH * SW * PXS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = a.tiles_x * a.tiles_y;
    const int b = blockIdx.x / per, tl = blockIdx.x - b * per;
    const int y0 = tl / a.tiles_x * TH, x0 = (tl - tl / a.tiles_x * a.tiles_x) * kTileX;
    const int h = a.h, w = a.w;

    // input tile
    constexpr int U = SH * SW * C8, LOADS = (U + 255) / 256;
    u32x4 v[LOADS];
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
        const int i = tid + l * 256, px = i / C8, c = (i - px * C8) * 8;
        const int sy = px / SW, sx = px - sy * SW, yy = y0 + sy - 1, xx = x0 + sx - 1;
        v[l] = u32x4{0u, 0u, 0u, 0u};
        if (i < U && yy >= 0 && yy < h && xx >= 0 && xx < w) {
            const bf16_t *src =
                c < C1 ? a.low + ((size_t)(b * (h / 2) + yy / 2) * (w / 2) + xx / 2) * C1 + c
                       : a.x + ((size_t)(b * h + yy) * w + xx) * (CIN - C1) + (c - C1);
            v[l] = *reinterpret_cast<const u32x4 *>(src);
        }
    }
    // the weights of the first steps, loaded while the tile arrives
    constexpr int PREW = HEAD ? 8 : 16 / NTW, PRE = PREW < STEPS ? PREW : STEPS;
    const int px = lane & 15, grp = lane >> 4;
    const int wn = wave % WN, row0 = wave / WN * NG;
    const bf16_t *wb = a.wgt + (size_t)(wn * NTW * 16 + px) * KPAD + grp * 8;
    u32x4 wpre[PRE][NTW];
#pragma unroll
    for (int s = 0; s < PRE; ++s)
#pragma unroll
        for (int t = 0; t < NTW; ++t)
            if (NT % WN == 0 || wn * NTW + t < NT)
                wpre[s][t] = *reinterpret_cast<const u32x4 *>(wb + (size_t)t * 16 * KPAD + 32 * s);
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
        const int i = tid + l * 256, px = i / C8, c = (i - px * C8) * 8;
        if (i < U) *reinterpret_cast<u32x4 *>(tile + px * PXS + c * 2) = v[l];
        if (C1 == 0 && a.xcopy) {  // the kept copy of the input: each tile its own pixels
            const int sy = px / SW, sx = px - sy * SW, yy = y0 + sy - 1, xx = x0 + sx - 1;
            if (i < U && sy >= 1 && sy <= TH && sx >= 1 && sx <= kTileX && yy < h && xx < w)
                *reinterpret_cast<u32x4 *>(a.xcopy + ((size_t)(b * h + yy) * w + xx) * CIN + c) = v[l];
        }
    }
    __syncthreads();

    f32x4 acc[NTW][NG];
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[t][g] = f32x4{0.f, 0.f, 0.f, 0.f};
    // what the end of the kernel reads, loaded here
    float qr[NG];
    u32x4 hw = {0u, 0u, 0u, 0u};
    f32x4 hb = {0.f, 0.f, 0.f, 0.f};
    if constexpr (HEAD) {
        hw = *reinterpret_cast<const u32x4 *>(a.head_w + px * 32 + grp * 8);
        hb = *reinterpret_cast<const f32x4 *>(a.head_b + 4 * grp);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int y = y0 + row0 + g, x = x0 + px;
            qr[g] = y < h && x < w ? a.q_ref[(size_t)(b * h + y) * w + x] : 1.f;
        }
    }
    const unsigned char *lb = tile + (row0 * SW + px) * PXS + (grp & 1) * 16;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        // lane groups 0, 1 hold channels k .. k + 15 of the step, groups 2, 3 the next 16: each within one tap
        const int kA = 32 * s, kB = kA + 16;
        const int tA = kA / CIN, tB = kB < K ? kB / CIN : 0;
        const int offA = (tA / 3 * SW + tA % 3) * PXS + (kA - tA * CIN) * 2;
        const int offB = kB < K ? (tB / 3 * SW + tB % 3) * PXS + (kB - tB * CIN) * 2 : 0;
        const int off = grp < 2 ? offA : offB;
        u32x4 bv[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            bv[g] = *reinterpret_cast<const u32x4 *>(lb + g * SW * PXS + off);
            if (kB >= K && grp >= 2) bv[g] = u32x4{0u, 0u, 0u, 0u};  // past the last tap
        }
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
            if (NT % WN != 0 && wn * NTW + t >= NT) continue;
            const u32x4 av =
                s < PRE ? wpre[s < PRE ? s : 0][t] : *reinterpret_cast<const u32x4 *>(wb + (size_t)t * 16 * KPAD + kA);
#pragma unroll
            for (int g = 0; g < NG; ++g)
                acc[t][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                                    __builtin_bit_cast(bf16x8, bv[g]), acc[t][g], 0, 0, 0);
        }
    }

    // acc[t][g][i]: output channel 16 (wn NTW + t) + 4 grp + i of pixel (x0 + px, y0 + row0 + g)
    const int x = x0 + px;
    if (HEAD) __syncthreads();  // the tile is read no more: each wave keeps its output rows there
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
        const int co = (wn * NTW + t) * 16 + 4 * grp;
        if (NT % WN != 0 && wn * NTW + t >= NT) continue;
        float bias[4] = {0.f, 0.f, 0.f, 0.f};
        if (a.bias) {
            const f32x4 bb = *reinterpret_cast<const f32x4 *>(a.bias + co);
#pragma unroll
            for (int i = 0; i < 4; ++i) bias[i] = bb[i];
        }
        float r[NG][4];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int y = y0 + row0 + g;
            const bool in = y < h && x < w;
            const size_t o = ((size_t)(b * h + y) * w + x) * COUT + co;
            u32x2 m = {0u, 0u};
            if (a.mask && in) m = *reinterpret_cast<const u32x2 *>(a.mask + o);
            bf16_t q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float u = acc[t][g][i] + bias[i];
                if (a.relu) u = fmaxf(u, 0.f);
                if (a.mask && !(bf2f((bf16_t)(m[i >> 1] >> (16 * (i & 1)))) > 0.f)) u = 0.f;
                q[i] = f2bf(u);
                r[g][i] = bf2f(q[i]);
            }
            const u32x2 st = {(uint32_t)q[0] | ((uint32_t)q[1] << 16), (uint32_t)q[2] | ((uint32_t)q[3] << 16)};
            if (in) *reinterpret_cast<u32x2 *>(a.y + o) = st;
            if (HEAD) *reinterpret_cast<u32x2 *>(tile + ((wave * NG + g) * 16 + px) * 48 + grp * 8) = st;
        }
        if constexpr (POOL) {
            // means of the stored values over 2 x 2 pixels: this lane's, the next lane's, then the row below
            float m[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float n0 = pair_swap(r[0][i]), n1 = pair_swap(r[1][i]);
                m[i] = ((((0.f + r[0][i]) + n0) + r[1][i]) + n1) * 0.25f;
            }
            const int y = y0 + row0;
            if ((px & 1) == 0 && y < h && x < w) {
                const u32x2 st = {(uint32_t)f2bf(m[0]) | ((uint32_t)f2bf(m[1]) << 16),
                                  (uint32_t)f2bf(m[2]) | ((uint32_t)f2bf(m[3]) << 16)};
                *reinterpret_cast<u32x2 *>(a.pool + ((size_t)(b * (h / 2) + y / 2) * (w / 2) + x / 2) * COUT + co) = st;
            }
        }
    }
    if constexpr (HEAD) {
        // the 1x1 head on the stored values: one MFMA, channels 16 .. 31 of its K zero
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            u32x4 dv = {0u, 0u, 0u, 0u};
            if (grp < 2) dv = *reinterpret_cast<const u32x4 *>(tile + ((wave * NG + g) * 16 + px) * 48 + grp * 16);
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, hw), __builtin_bit_cast(bf16x8, dv), z,
                                                        0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] += hb[i];
            const float z4 = __shfl(z[0], lane + 16, 64);  // lane group 1 holds outputs 4 .. 7
            const int y = y0 + row0 + g;
            if (y < h && x < w && grp < 2) {
                const size_t p = (size_t)(b * h + y) * w + x;
                *reinterpret_cast<f32x4 *>(a.z + p * kHeadPitch + 4 * grp) = z;
                if (grp == 0) {
                    a.q_copy[p] = qr[g];
                    if (a.out) {
                        const float nx = z[1], ny = z[2], nz = z[3];
                        const float inv = 1.f / __builtin_sqrtf(nx * nx + ny * ny + nz * nz);
                        float dq;
                        float *o = a.out + p * 5;
                        o[0] = 1.f / head_q(z[0], qr[g], a.dh, dq);
                        o[1] = nx * inv;
                        o[2] = ny * inv;
                        o[3] = nz * inv;
                        o[4] = sigmoidf(z4);
                    }
                }
            }
        }
    }
}

// Input gradient of the 1x1 head: g [P][16] (the loss's) x W' [16][32], masked by the layer below.
__global__ __launch_bounds__(256) void head_grad_kernel(const bf16_t *g, const bf16_t *wgt, const bf16_t *mask, int P,
                                                        bf16_t *out) {
    const int lane = threadIdx.x & 63, px = lane & 15, grp = lane >> 4;
    const long long p = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + px;
    const bool in = p < P;
    const u32x4 av = *reinterpret_cast<const u32x4 *>(wgt + px * 32 + grp * 8);
    u32x4 bv = {0u, 0u, 0u, 0u};
    if (in && grp < 2) bv = *reinterpret_cast<const u32x4 *>(g + p * 16 + grp * 8);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), acc, 0,
                                                  0, 0);
    if (!in) return;
    const u32x2 m = *reinterpret_cast<const u32x2 *>(mask + p * 16 + 4 * grp);
    bf16_t q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float u = acc[i] + 0.f;
        if (!(bf2f((bf16_t)(m[i >> 1] >> (16 * (i & 1)))) > 0.f)) u = 0.f;
        q[i] = f2bf(u);
    }
    *reinterpret_cast<u32x2 *>(out + p * 16 + 4 * grp) =
        u32x2{(uint32_t)q[0] | ((uint32_t)q[1] << 16), (uint32_t)q[2] | ((uint32_t)q[3] << 16)};
}

// ---------------------------------------------------------------------------
// Weight gradient: part[s][co][k] = sum over the pixels of split s of
// g[p][co] * x[p + offset(tap)][c], k = tap * cin + c;  bpart[s][co] = sum g[p][co].
//
// The product's K is the pixel, but memory holds a pixel's channels together:
// the operands come through the LDS transpose read (4 pixels x 16 channels per
// 16 lanes, each lane naming the pixel row it reads), so a tap's shift, the
// image borders and the split's end are only a choice of row -- a row of
// zeros where the tap falls outside.  A workgroup takes one split, one group
// of 16 input channels and one row of taps, a wave one tap and every output
// channel; blocks of B pixels are staged while the next one's loads are in
// flight (few workgroups: large blocks, so that few loads are waited for).  Sums run over 32 pixels per MFMA in pixel order, as before.
//
// Bound: LDS reads and the staging (a tap reads its 32 pixels x 16 channels
// once per MFMA), and in a split the chain of products.  16 x 120 x 160 cells,
// all layers: 12 launches with 16 two-byte loads per lane and MFMA took 1490
// us; staged, 195 us; a block's loads all in flight and their places advanced
// by carries (a division per unit and pixel before), 174 us.  (Not better:
// two blocks' loads in flight, the next round's operands read ahead -- the
// registers cost the second workgroup of a CU.)
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ s16x4 lds_read_tr(const bf16_t *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
}
__device__ __forceinline__ bf16x8 join8(s16x4 lo, s16x4 hi) {
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A pixel's place in the batch, advanced by a fixed step: carries instead of the divisions of its linear index.
struct Place {
    int x, y, b;
    __device__ __forceinline__ static Place of(int lin, int w, int h) {
        const int t = lin / w;
        return {lin - t * w, t % h, t / h};
    }
    __device__ __forceinline__ Place plus(const Place &d, int w, int h) const {
        Place r;
        r.x = x + d.x;
        const int cx = r.x >= w;
        r.x -= cx ? w : 0;
        r.y = y + d.y + cx;
        const int cy = r.y >= h;
        r.y -= cy ? h : 0;
        r.b = b + d.b + cy;
        return r;
    }
};

// NCO: output channels / 16; TAPS: 3 (3x3, blockIdx.z the row of taps) or 1 (1x1); B: pixels of a block.  The fourth
// wave (and with one tap the second and third) stages, and sums the bias gradient.
template <int NCO, int TAPS, int B>
__global__ __launch_bounds__(256) void wgrad_kernel(WgradArgs a) {
    constexpr int COUT = NCO * 16, NTHR = 256;
    constexpr int XU = (B + 2) * 2, GU = B * COUT / 8;                       // 16-byte units of a block
    constexpr int XL = (XU + NTHR - 1) / NTHR, GL = (GU + NTHR - 1) / NTHR;  // ... per thread
    __shared__ __align__(16) bf16_t xs[(B + 2 + 1) * 16];  // pixels lin0 .. lin0 + B + 1, and a row of zeros
    __shared__ __align__(16) bf16_t gs[B * COUT];
    __shared__ unsigned char flags[B];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = blockIdx.x, cg = blockIdx.y;
    const int dy = TAPS == 3 ? (int)blockIdx.z - 1 : 0, dx = TAPS == 3 ? wave - 1 : 0;
    const int w = a.w, h = a.h;
    const int P = a.n * h * w;
    const int beg = s * a.chunk, end = min(P, beg + a.chunk);
    // the channel group's source: the half-resolution one, or the other at its own channel offset
    const int c0 = cg * 16;
    const bool from_low = c0 < a.c1;
    const bf16_t *src = from_low ? a.low + c0 : a.x + (c0 - a.c1);
    const int cs = from_low ? a.c1 : a.cin - a.c1;  // channels of that source
    if (tid < 16) xs[(B + 2) * 16 + tid] = 0;

    // a block's places: of the thread's flags (pixels pb + tid, + NTHR, ...) and, where the source is the half-resolution
    // one, of its units (two to a pixel)
    const Place d_blk = Place::of(B, w, h), d_thr = Place::of(NTHR, w, h), d_unit = Place::of(NTHR / 2, w, h);
    Place fp = Place::of(beg + tid, w, h);
    // the units start up to w + 1 pixels before the split: two images are added and taken off again
    Place up = Place::of(beg + dy * w - 1 + (tid >> 1) + 2 * w * h, w, h);
    up.b -= 2;
    // no load is under a condition, so that all of a block are in flight: places outside the batch and pixels past the
    // split's end read its last ones (the flags send every tap of theirs to the row of zeros; g is cleared on its way to LDS)
    u32x4 xv[XL], gv[GL];
    const auto load = [&](int pb) {
        Place at = up;
#pragma unroll
        for (int l = 0; l < XL; ++l) {  // half a pixel's 16 channels each
            const int u = tid + l * NTHR;
            const int lin = pb + dy * w - 1 + (u >> 1);
            int q = min(max(lin, 0), P - 1);
            if (from_low) {
                q = min(max((at.b * (h / 2) + at.y / 2) * (w / 2) + at.x / 2, 0), P / 4 - 1);
                at = at.plus(d_unit, w, h);
            }
            xv[l] = *reinterpret_cast<const u32x4 *>(src + (size_t)q * cs + (u & 1) * 8);
        }
        if (from_low) up = up.plus(d_blk, w, h);
#pragma unroll
        for (int l = 0; l < GL; ++l) {
            const int u = tid + l * NTHR, q = min(pb + u / (COUT / 8), end - 1);
            gv[l] = *reinterpret_cast<const u32x4 *>(a.g + (size_t)q * COUT + (u % (COUT / 8)) * 8);
        }
    };
    load(beg);

    f32x4 acc[NCO];
    float bsum[NCO];
#pragma unroll
    for (int t = 0; t < NCO; ++t) {
        acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        bsum[t] = 0.f;
    }
    const bool do_bias = cg == 0 && blockIdx.z == 0 && wave == 3;
    // what a pixel must satisfy for this tap: inside the split, and the neighbour inside the image
    const int need = 16 | (dx < 0 ? 1 : dx > 0 ? 2 : 0) | (dy < 0 ? 4 : dy > 0 ? 8 : 0);
    const int l16 = lane & 15, grp = lane >> 4, sub = l16 >> 2, c4 = 4 * (l16 & 3);
    for (int pb = beg; pb < end; pb += B) {
        __syncthreads();  // the last block's reads
#pragma unroll
        for (int l = 0; l < XL; ++l)
            if (tid + l * NTHR < XU) *reinterpret_cast<u32x4 *>(xs + (tid + l * NTHR) * 8) = xv[l];
#pragma unroll
        for (int l = 0; l < GL; ++l)
            if (tid + l * NTHR < GU)
                *reinterpret_cast<u32x4 *>(gs + (tid + l * NTHR) * 8) =
                    pb + (tid + l * NTHR) / (COUT / 8) < end ? gv[l] : u32x4{0u, 0u, 0u, 0u};
        Place at = fp;
#pragma unroll
        for (int l = 0; l < B / NTHR; ++l) {
            const int i = tid + l * NTHR;
            flags[i] = (unsigned char)((at.x > 0 ? 1 : 0) | (at.x + 1 < w ? 2 : 0) | (at.y > 0 ? 4 : 0) |
                                       (at.y + 1 < h ? 8 : 0) | (pb + i < end ? 16 : 0));
            if (l + 1 < B / NTHR) at = at.plus(d_thr, w, h);
        }
        fp = fp.plus(d_blk, w, h);
        __syncthreads();
        if (pb + B < end) load(pb + B);
        // U steps together, so that their reads are in flight at once; those past the end meet zeros
        constexpr int U = NCO <= 2 ? 4 : 2;
        const int steps = (min(B, end - pb) + 31) / 32;
        if (wave < TAPS) {
            for (int st = 0; st < steps; st += U) {
                int r0[U], r1[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i0 = (st + u) * 32 + grp * 8 + sub;  // the lane's pixel rows: i0, i0 + 4
                    r0[u] = (flags[i0] & need) == need ? i0 + 1 + dx : B + 2;
                    r1[u] = (flags[i0 + 4] & need) == need ? i0 + 5 + dx : B + 2;
                }
                bf16x8 bx[U], ga[U][NCO];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i0 = (st + u) * 32 + grp * 8 + sub;
                    bx[u] = join8(lds_read_tr(xs + r0[u] * 16 + c4), lds_read_tr(xs + r1[u] * 16 + c4));
#pragma unroll
                    for (int t = 0; t < NCO; ++t)
                        ga[u][t] = join8(lds_read_tr(gs + i0 * COUT + t * 16 + c4),
                                         lds_read_tr(gs + (i0 + 4) * COUT + t * 16 + c4));
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int t = 0; t < NCO; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ga[u][t], bx[u], acc[t], 0, 0, 0);
            }
        } else if (do_bias) {
            // a lane's sum is a chain of additions in pixel order: the reads of V steps in flight (one step at a time it
            // added 10 us to the 9 us that staging 4800 pixels x 16 channels takes alone)
            constexpr int V = 4;
            for (int st = 0; st < steps; st += V) {
                s16x4 g[V][2][NCO];
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    const int i0 = (st + u) * 32 + grp * 8 + sub;
#pragma unroll
                    for (int t = 0; t < NCO; ++t) {
                        g[u][0][t] = lds_read_tr(gs + i0 * COUT + t * 16 + c4);
                        g[u][1][t] = lds_read_tr(gs + (i0 + 4) * COUT + t * 16 + c4);
                    }
                }
#pragma unroll
                for (int u = 0; u < V; ++u)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
#pragma unroll
                        for (int t = 0; t < NCO; ++t) bsum[t] += bf2f((bf16_t)g[u][e >> 2][t][e & 3]);
            }
        }
    }
    if (do_bias) {
#pragma unroll
        for (int t = 0; t < NCO; ++t) {
            bsum[t] += __shfl_xor(bsum[t], 16, 64);
            bsum[t] += __shfl_xor(bsum[t], 32, 64);
            if (grp == 0) a.bpart[(size_t)s * COUT + t * 16 + l16] = bsum[t];
        }
    }
    if (wave >= TAPS) return;
    // acc[t][i] = dW[16 t + 4 grp + i][tap cin + 16 cg + l16]
    const int tap = TAPS == 3 ? (dy + 1) * 3 + dx + 1 : 0;
    float *dst = a.part + (size_t)s * COUT * a.kpad + tap * a.cin + c0 + l16;
#pragma unroll
    for (int t = 0; t < NCO; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[(size_t)(t * 16 + 4 * grp + i) * a.kpad] = acc[t][i];
    }
}

// The gradient of every parameter from the splits' partial sums, in split order (one launch for the network; the
// loads of 16 splits are in flight together).  Padding gets 0.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(LayerTable tab, const float *part, int n_pad, float *grad) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n_pad) return;
    int li = 0;
    for (int l = 1; l < tab.n; ++l) li = e >= tab.l[l].w_off ? l : li;
    const LayerDims d = tab.l[li];
    const int n_w = d.cout_pad * d.kpad;
    const int o = e - d.w_off;
    bool live;
    const float *src;
    int stride;
    if (o < n_w) {
        live = o % d.kpad < d.taps * d.cin;
        src = part + (size_t)kMaxSplits * d.w_off + o;
        stride = n_w;
    } else {
        live = e - d.b_off < d.cout_pad;
        src = part + (size_t)kMaxSplits * d.b_off + (e - d.b_off);
        stride = d.cout_pad;
    }
    float sum = 0.f;
    if (live) {
        int k = 0;
        for (; k + 16 <= d.splits; k += 16) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = src[(size_t)(k + i) * stride];
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += v[i];
        }
        for (; k < d.splits; ++k) sum += src[(size_t)k * stride];
    }
    grad[e] = sum;
}

// Transposed, tap-mirrored weights of every layer for the input gradients, in one launch:
// W'[ci][tap' * cout_pad + co] = W[co][(taps - 1 - tap') * cin + ci]   (zero beyond taps * cout_pad)
__global__ __launch_bounds__(256) void transpose_w_kernel(LayerTable tab, const bf16_t *w, int n, bf16_t *wt) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    int li = 0;
    for (int l = 1; l < tab.n; ++l) li = e >= tab.l[l].t_off ? l : li;
    const LayerDims d = tab.l[li];
    const int o = e - d.t_off, ci = o / d.kpad_t, k = o - ci * d.kpad_t;
    bf16_t v = 0;
    if (ci < d.cin && k < d.taps * d.cout_pad) {
        const int tp = k / d.cout_pad, co = k - tp * d.cout_pad;
        v = w[d.w_off + (size_t)co * d.kpad + (d.taps - 1 - tp) * d.cin + ci];
    }
    wt[e] = v;
}

// ---------------------------------------------------------------------------
// gradients of the pooling and of the upsampling + concatenation (8 channels/thread)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void load8(const bf16_t *p, float v[8]) {
    const u32x4 u = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[2 * e] = bf2f((bf16_t)(u[e] & 0xffffu));
        v[2 * e + 1] = bf2f((bf16_t)(u[e] >> 16));
    }
}

__device__ __forceinline__ void store8(bf16_t *p, const float v[8]) {
    u32x4 u;
#pragma unroll
    for (int e = 0; e < 4; ++e) u[e] = (uint32_t)f2bf(v[2 * e]) | ((uint32_t)f2bf(v[2 * e + 1]) << 16);
    *reinterpret_cast<u32x4 *>(p) = u;
}

// gradient of an encoder output e that feeds both the pooling below and the
// decoder's concatenation:  g = (pool_grad(dp) + dcat[.., off + c]) * (e > 0)   (h, w: e's size)
__global__ void enc_grad_kernel(const bf16_t *dp, const bf16_t *dcat, int Ccat, int off, const bf16_t *e_act, int n,
                                int h, int w, int C, bf16_t *g) {
    const int C8 = C / 8;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * h * w * C8) return;
    const int c = (e % C8) * 8, q = e / C8;
    const int x = q % w, t = q / w, y = t % h, b = t / h;
    float a[8], d[8], m[8];
    load8(dp + ((size_t)(b * (h / 2) + y / 2) * (w / 2) + x / 2) * C + c, a);
    load8(dcat + (size_t)q * Ccat + off + c, d);
    load8(e_act + (size_t)q * C + c, m);
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = m[k] > 0.f ? fmaf(0.25f, a[k], d[k]) : 0.f;
    store8(g + (size_t)q * C + c, a);
}

// gradient of a low-resolution map upsampled into channels [0, C1) of a
// concatenation:  g = (sum over the 2 x 2 block of dcat) * (act > 0)   (h, w: low size)
__global__ void up_grad_kernel(const bf16_t *dcat, int Ccat, const bf16_t *act, int n, int h, int w, int C1,
                               bf16_t *g) {
    const int C8 = C1 / 8;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * h * w * C8) return;
    const int c = (e % C8) * 8, q = e / C8;
    const int j = q % w, t = q / w, i = t % h, b = t / h;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0}, v[8], m[8];
    for (int dy = 0; dy < 2; ++dy)
        for (int dx = 0; dx < 2; ++dx) {
            load8(dcat + ((size_t)(b * 2 * h + 2 * i + dy) * 2 * w + 2 * j + dx) * Ccat + c, v);
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] += v[k];
        }
    load8(act + (size_t)q * C1 + c, m);
#pragma unroll
    for (int k = 0; k < 8; ++k) s[k] = m[k] > 0.f ? s[k] : 0.f;
    store8(g + (size_t)q * C1 + c, s);
}

// ---------------------------------------------------------------------------
// loss and its gradient
// ---------------------------------------------------------------------------
// per pixel: w (|s - t_d| + 1 - n_hat . n_t) + softplus(z4) - t_c z4, and dL/dz / P
__global__ __launch_bounds__(256) void loss_kernel(const float *z, const float *q_ref, const float *target, int P,
                                                   DepthHead dh, bf16_t *dz, float *part) {
    __shared__ float red[256];
    const int p = blockIdx.x * 256 + threadIdx.x;
    float L = 0.f;
    if (p < P) {
        const float *zp = z + (size_t)p * kHeadPitch;
        const float *tp = target + (size_t)p * 6;
        const float invP = 1.f / (float)P;
        const float span = dh.d_max - dh.d_min;
        float dq;
        const float q = head_q(zp[0], q_ref[p], dh, dq);
        const float s = (1.f / q - dh.d_min) / span;
        const float td = (tp[0] - dh.d_min) / span;
        const float wdn = tp[5];
        const float nx = zp[1], ny = zp[2], nz = zp[3];
        const float nn = __builtin_sqrtf(nx * nx + ny * ny + nz * nz);
        const float inv = 1.f / nn;
        const float hx = nx * inv, hy = ny * inv, hz = nz * inv;
        const float cosang = hx * tp[1] + hy * tp[2] + hz * tp[3];
        const float z4 = zp[4], tc = tp[4];
        const float softplus = fmaxf(z4, 0.f) + __logf(1.f + __expf(-fabsf(z4)));
        const float diff = s - td;
        L = wdn * (fabsf(diff) + 1.f - cosang) + softplus - tc * z4;
        float g[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) g[k] = 0.f;
        const float sg = diff > 0.f ? 1.f : (diff < 0.f ? -1.f : 0.f);
        g[0] = wdn * sg * (-1.f / (q * q * span)) * dq * invP;
        const float wn = -wdn * inv * invP;
        g[1] = wn * (tp[1] - cosang * hx);
        g[2] = wn * (tp[2] - cosang * hy);
        g[3] = wn * (tp[3] - cosang * hz);
        g[4] = (sigmoidf(z4) - tc) * invP;
        store8(dz + (size_t)p * 16, g);
        store8(dz + (size_t)p * 16 + 8, g + 8);
    }
    red[threadIdx.x] = L;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// sum of the per-block loss partials in a fixed order, divided by P
__global__ void loss_reduce_kernel(const float *part, int n, int P, float *loss) {
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = (float)(red[0] / (double)P);
}

// ---------------------------------------------------------------------------
// Adam (Kingma & Ba) on the fp32 master parameters; refreshes the bf16 copy
// ---------------------------------------------------------------------------
__global__ void adam_kernel(float *p, const float *g, float *m, float *v, bf16_t *pb, int n, float lr, float b1,
                            float b2, float eps, float c1, float c2) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const float ge = g[e];
    const float me = b1 * m[e] + (1.f - b1) * ge;
    const float ve = b2 * v[e] + (1.f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    const float pe = p[e] - lr * (me / c1) / (__builtin_sqrtf(ve / c2) + eps);
    p[e] = pe;
    pb[e] = f2bf(pe);
}

// Training targets at the cell pixels (min(s j + s/2, W - 1), min(s i + s/2, H - 1)) of the network's grid of
// s x s cells: depth,
// normal, and the confidence C(m) = exp(-m^2 / (2 beta^2)) of Eq. 3 on the final matching cost m, twice (the
// confidence target and the weight of the depth and normal terms).
__global__ void targets_kernel(const float *depth, const float *normal, const float *cost, int W, int H, int cell,
                               int h4, int w4, float inv_2b2, float *target) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= h4 * w4) return;
    const int i = c / w4, j = c - i * w4;
    const int x = min(cell * j + cell / 2, W - 1), y = min(cell * i + cell / 2, H - 1);
    const size_t p = (size_t)y * W + x;
    const float m = cost[p];
    const float conf = expf(-m * m * inv_2b2);
    float *t = target + (size_t)c * 6;
    t[0] = depth[p];
    t[1] = normal[3 * p];
    t[2] = normal[3 * p + 1];
    t[3] = normal[3 * p + 2];
    t[4] = conf;
    t[5] = conf;
}

hipError_t launch_targets(const float *depth, const float *normal, const float *cost, int W, int H, int cell,
                          int h4, int w4, float beta, float *target, hipStream_t s) {
    const int n = h4 * w4;
    hipLaunchKernelGGL(targets_kernel, dim3((n + 255) / 256), dim3(256), 0, s, depth, normal, cost, W, H, cell, h4,
                       w4, 1.f / (2.f * beta * beta), target);
    return hipGetLastError();
}

__global__ void to_bf16_kernel(const float *src, int n, bf16_t *dst) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) dst[e] = f2bf(src[e]);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline dim3 grid1(long long n, int bs = 256) { return dim3((unsigned)((n + bs - 1) / bs)); }

template <int CIN, int COUT, int C1, int WN, int NG, bool POOL = false, bool HEAD = false>
static hipError_t run_conv3(Conv3Args a, hipStream_t s) {
    constexpr int TH = 4 / WN * NG;
    a.tiles_x = (a.w + kTileX - 1) / kTileX;
    a.tiles_y = (a.h + TH - 1) / TH;
    const long long blocks = (long long)a.n * a.tiles_x * a.tiles_y;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffll) return hipErrorInvalidValue;
    NN_LAUNCH((conv3_kernel<CIN, COUT, C1, WN, NG, POOL, HEAD>), dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Tile shapes, by layer (each layer works at one resolution), as measured at 320 x 480 cells: two rows per wave (8-row
// tiles) on the upper levels; on the quarter- and eighth-resolution levels, whose few pixels would leave CUs idle there, one
// row per wave or waves split over the output channels.  The image's size doesn't enter.
hipError_t launch_conv3(int cin, int cout, const Conv3Args &a, hipStream_t s) {
    if (a.head_w) return cin == 48 && cout == 16 && a.low ? run_conv3<48, 16, 32, 1, 2, false, true>(a, s) : hipErrorInvalidValue;
    if (a.low) {
        if (cin == 112 && cout == 48) return run_conv3<112, 48, 64, 4, 2>(a, s);
        if (cin == 80 && cout == 32) return run_conv3<80, 32, 48, 2, 2>(a, s);
        return hipErrorInvalidValue;
    }
    if (a.pool) {
        if (cin == 16 && cout == 16) return run_conv3<16, 16, 0, 1, 2, true>(a, s);
        if (cin == 32 && cout == 32) return run_conv3<32, 32, 0, 1, 2, true>(a, s);
        if (cin == 48 && cout == 48) return run_conv3<48, 48, 0, 4, 2, true>(a, s);
        return hipErrorInvalidValue;
    }
    if (cin == 16) {
        if (cout == 16) return run_conv3<16, 16, 0, 1, 2>(a, s);
        if (cout == 32) return run_conv3<16, 32, 0, 1, 2>(a, s);
        if (cout == 48) return run_conv3<16, 48, 0, 1, 2>(a, s);
    } else if (cin == 32) {
        if (cout == 16) return run_conv3<32, 16, 0, 1, 2>(a, s);
        if (cout == 32) return run_conv3<32, 32, 0, 1, 2>(a, s);
        if (cout == 48) return run_conv3<32, 48, 0, 1, 1>(a, s);
        if (cout == 80) return run_conv3<32, 80, 0, 1, 2>(a, s);
    } else if (cin == 48) {
        if (cout == 32) return run_conv3<48, 32, 0, 1, 1>(a, s);
        if (cout == 48) return run_conv3<48, 48, 0, 1, 1>(a, s);
        if (cout == 64) return run_conv3<48, 64, 0, 4, 2>(a, s);
        if (cout == 112) return run_conv3<48, 112, 0, 1, 1>(a, s);
    } else if (cin == 64) {
        if (cout == 48) return run_conv3<64, 48, 0, 1, 1>(a, s);
        if (cout == 64) return run_conv3<64, 64, 0, 4, 2>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_head_grad(const bf16_t *g, const bf16_t *wgt, const bf16_t *mask, int P, bf16_t *out, hipStream_t s) {
    NN_LAUNCH(head_grad_kernel, grid1(P, 64), dim3(256), 0, s, g, wgt, mask, P, out);
    return hipGetLastError();
}

hipError_t launch_wgrad(const WgradArgs &a, int splits, hipStream_t s) {
    const dim3 grid(splits, a.cin / 16, a.ks);
    if (a.ks == 1) {
        if (a.cout_pad != 16) return hipErrorInvalidValue;
        NN_LAUNCH((wgrad_kernel<1, 1, 1024>), grid, dim3(256), 0, s, a);
        return hipGetLastError();
    }
    switch (a.cout_pad / 16) {  // 33, 50, 33 and 41 KB of LDS (67 KB for the 1x1 head above)
        case 1: NN_LAUNCH((wgrad_kernel<1, 3, 512>), grid, dim3(256), 0, s, a); break;
        case 2: NN_LAUNCH((wgrad_kernel<2, 3, 512>), grid, dim3(256), 0, s, a); break;
        case 3: NN_LAUNCH((wgrad_kernel<3, 3, 256>), grid, dim3(256), 0, s, a); break;
        case 4: NN_LAUNCH((wgrad_kernel<4, 3, 256>), grid, dim3(256), 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const LayerTable &tab, const float *part, int n_pad, float *grad, hipStream_t s) {
    NN_LAUNCH(wgrad_reduce_kernel, grid1(n_pad), dim3(256), 0, s, tab, part, n_pad, grad);
    return hipGetLastError();
}

hipError_t launch_transpose_w(const LayerTable &tab, const bf16_t *w, int n, bf16_t *wt, hipStream_t s) {
    NN_LAUNCH(transpose_w_kernel, grid1(n), dim3(256), 0, s, tab, w, n, wt);
    return hipGetLastError();
}

hipError_t launch_enc_grad(const bf16_t *dp, const bf16_t *dcat, int Ccat, int off, const bf16_t *e_act, int n, int h,
                           int w, int C, bf16_t *g, hipStream_t s) {
    NN_LAUNCH(enc_grad_kernel, grid1((long long)n * h * w * (C / 8)), dim3(256), 0, s, dp, dcat, Ccat, off, e_act, n,
              h, w, C, g);
    return hipGetLastError();
}

hipError_t launch_up_grad(const bf16_t *dcat, int Ccat, const bf16_t *act, int n, int h, int w, int C1, bf16_t *g,
                          hipStream_t s) {
    NN_LAUNCH(up_grad_kernel, grid1((long long)n * h * w * (C1 / 8)), dim3(256), 0, s, dcat, Ccat, act, n, h, w, C1,
              g);
    return hipGetLastError();
}

int loss_blocks(int P) { return (P + 255) / 256; }

hipError_t launch_loss(const float *z, const float *q_ref, const float *target, int P, const DepthHead &dh, bf16_t *dz,
                       float *part, float *loss, hipStream_t s) {
    const int nb = loss_blocks(P);
    NN_LAUNCH(loss_kernel, dim3(nb), dim3(256), 0, s, z, q_ref, target, P, dh, dz, part);
    NN_LAUNCH(loss_reduce_kernel, dim3(1), dim3(256), 0, s, part, nb, P, loss);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, bf16_t *pb, int n, float lr, float b1, float b2,
                       float eps, int step, hipStream_t s) {
    const float c1 = 1.f - (float)std::pow((double)b1, (double)step);
    const float c2 = 1.f - (float)std::pow((double)b2, (double)step);
    NN_LAUNCH(adam_kernel, grid1(n), dim3(256), 0, s, p, g, m, v, pb, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *src, int n, bf16_t *dst, hipStream_t s) {
    NN_LAUNCH(to_bf16_kernel, grid1(n), dim3(256), 0, s, src, n, dst);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace amh
