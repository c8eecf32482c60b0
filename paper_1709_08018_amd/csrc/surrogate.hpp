// surrogate.hpp -- declarations shared by the surrogate's inference kernels
// (surrogate.hip) and its training kernels (surrogate_train.hip): the layout
// of the parameter vector and of the workspace, and the matrix-core helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "kl_internal.hpp"
#include "kl_surrogate.h"

namespace kl {
namespace sur {

typedef unsigned short bf16_t;
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kImg = KL_SUR_IMG;

// parameter layout (offsets in floats)
struct Layout {
    size_t W1, b1, W2, b2, K1, c1, K2, c2, K3, c3, K4, c4, total;
};
inline Layout layout() {
    Layout L;
    size_t o = 0;
    L.W1 = o; o += 4 * 256;
    L.b1 = o; o += 256;
    L.W2 = o; o += 256 * 256;
    L.b2 = o; o += 256;
    L.K1 = o; o += 16 * 64 * 16;
    L.c1 = o; o += 64;
    L.K2 = o; o += 64 * 32 * 16;
    L.c2 = o; o += 32;
    L.K3 = o; o += 32 * 16 * 16;
    L.c3 = o; o += 16;
    L.K4 = o; o += 16 * 1 * 16;
    L.c4 = o; o += 1;
    L.total = o;
    return L;
}

// FP32 -> bfloat16, round to nearest even
__device__ __forceinline__ bf16_t to_bf16(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// the value of x rounded to bfloat16, as FP32
__device__ __forceinline__ float bf16_value(float x) { return __uint_as_float((uint32_t)to_bf16(x) << 16); }

// D = A B + C on the matrix cores, one wave.  A (16 x K): lane l holds row
// l % 16, K / 4 consecutive k from (K / 4) (l / 16); B (K x 16) likewise by
// column; D (16 x 16): lane l holds column l % 16, rows 4 (l / 16) .. + 3.
__device__ __forceinline__ f32x4 mma16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma32(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Stride-2, pad-1 transposed convolution: for output phase p (0 even, 1
// odd) and tap a (0, 1), the input offset and kernel index.
__device__ __forceinline__ int tap_dy(int p, int a) { return p ? (a ? 0 : 1) : (a ? -1 : 0); }
__device__ __forceinline__ int tap_k(int p, int a) { return p ? (a ? 2 : 0) : (a ? 3 : 1); }

// Packed bfloat16 weights (offsets in elements), rounded once a pass into
// operand order: a fragment is the 64 lanes' values one after another (lane
// l's row l % 16 and its 4, or for mma32 8, consecutive k from l / 16), so that
// a wave reads it as one contiguous piece.  Read from the parameters' own
// order a fragment is 64 separate requests, some 60 cycles of a CU's address
// unit each: the weights of the second layer's backward alone took 7 us.
constexpr int kT1f = 0;                       // K1 forward: [tap][o / 16], k = c
constexpr int kT4f = kT1f + 16 * 64 * 16;     // K4 forward: rows taps, k = c
constexpr int kI2 = kT4f + 16 * 16;           // K2 forward, mma32: [phase][tap][c / 32][o / 16], k = c % 32
constexpr int kI3 = kI2 + 16 * 32 * 64;       // K3 forward, mma32: [phase][tap], k = c
constexpr int kForwardPacked = kI3 + 16 * 16 * 32;
constexpr int kT2f = kForwardPacked;          // K2 forward: [phase][tap][o / 16][c / 16]
constexpr int kT3f = kT2f + 16 * 32 * 64;     // K3 forward: [phase][tap][c / 16]
constexpr int kT1b = kT3f + 16 * 16 * 32;     // K1 backward: [o], rows c, k = taps
constexpr int kT2b = kT1b + 16 * 64 * 16;     // K2 backward: [c / 16][o], k = taps
constexpr int kT3b = kT2b + 64 * 32 * 16;     // K3 backward: [c / 16][o]
constexpr int kT4b = kT3b + 32 * 16 * 16;     // K4 backward: rows c, k = taps
constexpr int kT2w = kT4b + 16 * 16;          // W2 backward: [i / 16][j / 16], rows i, k = j
constexpr int kTrainPacked = kT2w + 256 * 256;

// Packed element e of the parameters P.
__device__ __forceinline__ float packed_weight(const float* P, const Layout& L, int e) {
    auto taps = [](int ph, int tap) { return tap_k(ph >> 1, tap >> 1) * 4 + tap_k(ph & 1, tap & 1); };
    if (e >= kI2 && e < kForwardPacked) {   // mma32 fragments
        const int i = (e - kI2) % 512, f = (e - kI2) / 512, row = i / 8 % 16, k = 8 * (i / 128) + i % 8;
        if (e < kI3) {
            const int o = 16 * (f % 2) + row, c = 32 * (f / 2 % 2) + k, tap = f / 4 % 4, ph = f / 16;
            return P[L.K2 + (c * 32 + o) * 16 + taps(ph, tap)];
        }
        const int g = (e - kI3) / 512;
        return P[L.K3 + (k * 16 + row) * 16 + taps(g / 4, g % 4)];
    }
    const int row = e / 4 % 16, k = 4 * (e / 64 % 4) + e % 4;   // every offset is a multiple of a fragment's 256
    if (e < kT4f) {
        const int f = e / 256;
        return P[L.K1 + (k * 64 + 16 * (f % 4) + row) * 16 + f / 4];
    }
    if (e < kI2) return P[L.K4 + k * 16 + row];
    if (e < kT3f) {
        const int f = (e - kT2f) / 256, c = 16 * (f % 4) + k, o = 16 * (f / 4 % 2) + row;
        return P[L.K2 + (c * 32 + o) * 16 + taps(f / 32, f / 8 % 4)];
    }
    if (e < kT1b) {
        const int f = (e - kT3f) / 256, c = 16 * (f % 2) + k;
        return P[L.K3 + (c * 16 + row) * 16 + taps(f / 8, f / 2 % 4)];
    }
    if (e < kT2b) return P[L.K1 + (row * 64 + (e - kT1b) / 256) * 16 + k];
    if (e < kT3b) {
        const int f = (e - kT2b) / 256;
        return P[L.K2 + ((16 * (f / 32) + row) * 32 + f % 32) * 16 + k];
    }
    if (e < kT4b) {
        const int f = (e - kT3b) / 256;
        return P[L.K3 + ((16 * (f / 16) + row) * 16 + f % 16) * 16 + k];
    }
    if (e < kT2w) return P[L.K4 + row * 16 + k];
    const int f = (e - kT2w) / 256;
    return P[L.W2 + (16 * (f / 16) + row) * 256 + 16 * (f % 16) + k];
}

// Vectors of global memory, 4-byte aligned: callers may pass any float array
typedef float f32x4g __attribute__((ext_vector_type(4), aligned(4)));
typedef short bf16x4g __attribute__((ext_vector_type(4), aligned(4)));
typedef short bf16x8g __attribute__((ext_vector_type(8), aligned(4)));

__device__ __forceinline__ f32x4 load4(const float* p) { return *(const f32x4g*)p; }
__device__ __forceinline__ void store4(float* p, f32x4 v) { *(f32x4g*)p = v; }
__device__ __forceinline__ bf16x4 loadw(const bf16_t* p) { return *(const bf16x4g*)p; }
// fragment f of packed weights, this lane's part
__device__ __forceinline__ bf16x4 frag4(const bf16_t* w, int f, int lane) { return *(const bf16x4g*)(w + (f * 64 + lane) * 4); }
__device__ __forceinline__ bf16x8 frag8(const bf16_t* w, int f, int lane) { return *(const bf16x8g*)(w + (f * 64 + lane) * 8); }
__device__ __forceinline__ bf16x4 lds4(const bf16_t* p) { return *(const bf16x4*)p; }   // 8-byte aligned LDS
__device__ __forceinline__ bf16x8 lds8(const bf16_t* p) { return *(const bf16x8*)p; }   // 16-byte aligned LDS

// two values rounded to bfloat16 (nearest even): v_cvt_pk_bf16_f32, one
// instruction where to_bf16's integer form takes ten
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bfloat2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bfloat2));
}
__device__ __forceinline__ bf16x4 round4(f32x4 v) {
    const uint2 u = {pack2(v[0], v[1]), pack2(v[2], v[3])};
    return __builtin_bit_cast(bf16x4, u);
}

constexpr f32x4 kZero4 = {0.f, 0.f, 0.f, 0.f};

__device__ __forceinline__ f32x4 add4(f32x4 a, f32x4 b) { return a + b; }
__device__ __forceinline__ f32x4 relu4(f32x4 a) {
    return f32x4{fmaxf(a[0], 0.f), fmaxf(a[1], 0.f), fmaxf(a[2], 0.f), fmaxf(a[3], 0.f)};
}

// One Adam update (bc: the step's bias corrections), by its own kernel or at
// the end of a training step.  p == nullptr: none.
struct Adam {
    float *p, *m, *v;
    float lr, bc1, bc2;
    __device__ __forceinline__ void update(int64_t e, float g) const {
        const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
        const float me = b1 * m[e] + (1.f - b1) * g;
        const float ve = b2 * v[e] + (1.f - b2) * g * g;
        m[e] = me;
        v[e] = ve;
        p[e] -= lr * (me / bc1) / (sqrtf(ve / bc2) + eps);
    }
};

// Workgroups of the training kernels that keep a weight gradient in their
// registers over several sets, each leaving one partial sum.
constexpr int kParts3 = 512, kParts2 = 64, kParts1 = 128;
// floats of one workgroup's partial sums: the last two layers' (loss, bias 4,
// bias 3 at 2 .. 17, K4 at 32 .. 287), and K3 with bias 2
constexpr int kPart34 = 288, kPart3 = 32 * 256 + 32, kPart2 = 64 * 512, kPart1 = 16 * 1024;

struct WS {
    float *u, *h1, *h2, *x0, *y1, *y2, *y3, *logits, *dlogits, *dy3, *dy2, *dy1, *dx0, *dh2, *dh1;
    // partial sums: last two layers (8 a set), K3 and bias 2, bias 1 (2 a set, 64 each), K2, K1
    float *p34, *p3, *pc1, *p2, *p1;
    bf16_t* packed;   // packed weights of one pass, forward or training
    bf16_t* x0h;      // the inference path's input of the first transposed convolution: b x 16 pixels x 16 channels
    size_t bytes;
};

WS carve(void* base, int B);

hipError_t loss_grad(const float* P, const kl_c64* ta, const kl_c64* tb, const uint8_t* targets, int B, float* G,
                     float* loss, const Adam& adam, const WS& w, hipStream_t s);

}  // namespace sur
}  // namespace kl
