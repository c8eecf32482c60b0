// surrogate.hip -- inference kernels of the occupancy surrogate
// (include/kl_surrogate.h), its optimiser, gate and IoU kernels, the BF16
// matrix-core GEMM with FP32 accumulation, and the entry points.  A training
// step's loss and gradient are in surrogate_train.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "surrogate.hpp"

namespace kl {
namespace sur {

// ------------------------------------------------------------------ GEMM
struct GemmArgs {
    int M, N, K;
    const float* A;
    int64_t lam, lak;
    const float* B;
    int64_t lbk, lbn;
    float* C;
    int64_t ldc;
    const float* bias;
    int relu, accumulate, ksplit, kchunk;
};

constexpr int kTM = 64, kTN = 64, kTK = 32, kPad = 8;

// 256 threads: 4 waves in a 2 x 2 arrangement of 32 x 32 wave tiles, each
// 2 x 2 MFMA 16x16x16 tiles.  A and B tiles are staged in LDS as bfloat16
// (B transposed, so both fragments are 4 consecutive k of one row).
// With ksplit > 1 each z-slice of the grid sums one chunk of K and adds it
// to C atomically.
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const GemmArgs g) {
    __shared__ unsigned short As[kTM][kTK + kPad];
    __shared__ unsigned short Bs[kTN][kTK + kPad];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int bm = blockIdx.y * kTM, bn = blockIdx.x * kTN;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int kbeg = blockIdx.z * g.kchunk;
    const int kend = std::min(g.K, kbeg + g.kchunk);
    f32x4 acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = kbeg; k0 < kend; k0 += kTK) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = tid * 8 + u;
            const int r = e / kTK, k = e % kTK;   // A tile: 64 rows x 32 k
            const int gi = bm + r, gk = k0 + k;
            float va = 0.f;
            if (gi < g.M && gk < kend) va = g.A[(int64_t)gi * g.lam + (int64_t)gk * g.lak];
            As[r][k] = to_bf16(va);
            const int kb = e / kTN, c = e % kTN;  // B tile: 32 k x 64 cols
            const int gj = bn + c, gkb = k0 + kb;
            float vb = 0.f;
            if (gj < g.N && gkb < kend) vb = g.B[(int64_t)gkb * g.lbk + (int64_t)gj * g.lbn];
            Bs[c][kb] = to_bf16(vb);
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kTK; ks += 16) {
            bf16x4 af[2], bfr[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const unsigned short* pa = &As[wm + t * 16 + (lane & 15)][ks + 4 * (lane >> 4)];
                const unsigned short* pb = &Bs[wn + t * 16 + (lane & 15)][ks + 4 * (lane >> 4)];
                af[t] = bf16x4{(short)pa[0], (short)pa[1], (short)pa[2], (short)pa[3]};
                bfr[t] = bf16x4{(short)pb[0], (short)pb[1], (short)pb[2], (short)pb[3]};
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af[a], bfr[b], acc[a][b], 0, 0, 0);
        }
        __syncthreads();
    }
    // D(i, j): lane holds column (lane & 15), rows 4 * (lane >> 4) + v
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = bm + wm + a * 16 + 4 * (lane >> 4) + v;
                const int j = bn + wn + b * 16 + (lane & 15);
                if (i >= g.M || j >= g.N) continue;
                float x = acc[a][b][v];
                float* dst = g.C + (int64_t)i * g.ldc + j;
                if (g.ksplit > 1) {
                    atomicAdd(dst, x);
                } else if (g.accumulate) {
                    *dst += x;
                } else {
                    if (g.bias) x += g.bias[j];
                    if (g.relu) x = fmaxf(x, 0.f);
                    *dst = x;
                }
            }
}

__global__ void zero_rows_kernel(float* C, int M, int N, int64_t ldc) {
    const int64_t n = (int64_t)M * N;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        C[(e / N) * ldc + (e % N)] = 0.f;
}

static hipError_t gemm(int M, int N, int K, const float* A, int64_t lam, int64_t lak, const float* B, int64_t lbk,
                       int64_t lbn, float* C, int64_t ldc, const float* bias, int relu, int accumulate,
                       hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    GemmArgs g{M, N, K, A, lam, lak, B, lbk, lbn, C, ldc, bias, relu, accumulate, 1, 0};
    const int tiles = ((M + kTM - 1) / kTM) * ((N + kTN - 1) / kTN);
    int ksplit = 1;
    // few output tiles and a long K: spread K over more workgroups
    if (!bias && !relu && tiles < 512 && K > 4 * kTK) {
        ksplit = std::min((K + 4 * kTK - 1) / (4 * kTK), std::max(1, 1024 / tiles));
    }
    int chunk = (K + ksplit - 1) / ksplit;
    chunk = ((chunk + kTK - 1) / kTK) * kTK;
    if (chunk < kTK) chunk = kTK;
    ksplit = std::max(1, (K + chunk - 1) / chunk);
    g.ksplit = ksplit;
    g.kchunk = K > 0 ? chunk : kTK;
    if (ksplit > 1 && !accumulate) {
        hipLaunchKernelGGL(zero_rows_kernel, dim3(std::min<int64_t>(4096, ((int64_t)M * N + 255) / 256)), dim3(256),
                           0, s, C, M, N, ldc);
    }
    if (K <= 0) return hipGetLastError();
    dim3 grid((N + kTN - 1) / kTN, (M + kTM - 1) / kTM, ksplit);
    hipLaunchKernelGGL(gemm_bf16_kernel, grid, dim3(256), 0, s, g);
    return hipGetLastError();
}

__global__ void adam_kernel(const Adam a, const float* g, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        a.update(e, g[e]);
}

__global__ void occupancy_kernel(const uint32_t* c, uint64_t n, uint8_t* o) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (uint64_t)gridDim.x * blockDim.x)
        o[e] = c[e] > 0u ? 1 : 0;
}

__global__ void predict_occupancy_kernel(const float* z, uint64_t n, uint8_t* o) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (uint64_t)gridDim.x * blockDim.x)
        o[e] = z[e] > 0.f ? 1 : 0;
}

// One workgroup per set: mean binary entropy of sigmoid(z).  Bound by its
// arithmetic (8.4 M logits at 512 sets), so a set takes sixteen waves, which
// fill a CU's schedulers at two sets a CU, and a logit one exponential and
// one reciprocal: with e = e^-|x| and s = e / (2 + e),
//   H(sigmoid(x)) = log(1 + e) + |x| e / (1 + e),   log(1 + e) = 2 atanh(s),
// the atanh by its power series to s^15 (s <= 1/3: truncated below 2e-9 of
// its value).  512 sets: 10.9 us; with four waves a set, log1pf, and a
// second exponential 43 us, with sixteen waves and log1pf 27 us.
__device__ __forceinline__ float binary_entropy(float x) {
    const float a = fabsf(x), e = expf(-a), p = 1.f + e, q = 2.f + e, pq = p * q;
    float r = __builtin_amdgcn_rcpf(pq);   // 2 <= pq <= 6; one Newton step to full precision
    r = fmaf(r, fmaf(-pq, r, 1.f), r);
    const float s = e * (p * r), z = s * s;
    float c = 1.f / 15.f;
    c = fmaf(c, z, 1.f / 13.f);
    c = fmaf(c, z, 1.f / 11.f);
    c = fmaf(c, z, 1.f / 9.f);
    c = fmaf(c, z, 1.f / 7.f);
    c = fmaf(c, z, 1.f / 5.f);
    c = fmaf(c, z, 1.f / 3.f);
    return fmaf(2.f * s, c * z, 2.f * s) + a * (e * (q * r));
}

constexpr int kUncThreads = 1024;

__global__ __launch_bounds__(kUncThreads) void uncertainty_kernel(const float* __restrict__ z, float* __restrict__ out) {
    __shared__ float red[kUncThreads / 64];
    const float* zs = z + (int64_t)blockIdx.x * kImg * kImg;
    float acc = 0.f;
#pragma unroll
    for (int q = 0; q < kImg * kImg / (4 * kUncThreads); ++q) {
        const f32x4 x = load4(zs + 4 * (q * kUncThreads + (int)threadIdx.x));
#pragma unroll
        for (int v = 0; v < 4; ++v) acc += binary_entropy(x[v]);
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float sum = 0.f;
        for (int w = 0; w < kUncThreads / 64; ++w) sum += red[w];
        out[blockIdx.x] = sum / (float)(kImg * kImg);
    }
}

__global__ void iou_kernel(const float* __restrict__ z, const uint8_t* __restrict__ pred,
                           const uint8_t* __restrict__ t, float* __restrict__ out) {
    __shared__ int ri[256], ru[256];
    const int64_t base = (int64_t)blockIdx.x * kImg * kImg;
    int inter = 0, uni = 0;
    for (int e = threadIdx.x; e < kImg * kImg; e += 256) {
        const bool p = z ? (z[base + e] > 0.f) : (pred[base + e] != 0);
        const bool q = t[base + e] != 0;
        inter += p && q;
        uni += p || q;
    }
    ri[threadIdx.x] = inter;
    ru[threadIdx.x] = uni;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            ri[threadIdx.x] += ri[threadIdx.x + w];
            ru[threadIdx.x] += ru[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = ru[0] == 0 ? 1.f : (float)ri[0] / (float)ru[0];
}

// ------------------------------------------------------------------ forward (inference)
// Two launches, activations in LDS as bfloat16 -- the rounding the training
// path applies when it reads them as product operands.
//
// forward_mlp_kernel: the linear layers of 16 sets a workgroup (u -> h1, four
// products per output on the vector ALUs; h1 -> h2 on the matrix cores, the
// sets in the columns), and in further workgroups the packed weights.
//
// forward_kernel: the transposed convolutions of one set's strip of 32 logit
// rows (y3 rows 16 s - 1 .. 16 s + 16, y2 rows 8 s - 1 .. 8 s + 8, y1 rows
// 4 s - 1 .. 4 s + 4; a neighbour's rows are formed again, 1.2 times the
// products of a whole set):
//   * convT k4 s4 p0 (16 -> 64 channels, 4^2 -> 16^2): one product per tap
//     and 16 channels, K1 by the 16 input pixels;
//   * convT k4 s2 p1: output pixel (2m + py, 2n + px) gathers the input
//     pixels (m + dy, n + dx) over two row taps and two column taps fixed by
//     the phase (py, px) (tap_dy, tap_k), so each of the four phases is a
//     2 x 2 convolution: Cout x (4 taps * Cin) weights times (4 taps * Cin) x
//     (16 pixels) read straight from the padded input in LDS, one tap and 32
//     channels per product step.  Taken this way round, a lane ends up
//     holding four consecutive channels of one output pixel;
//   * the last layer (16 -> 1 channel) in column form: col = y3 K4 (16 taps
//     per pixel).  A lane's four channels of y3 are exactly its operand of
//     that product, so y3 never leaves the registers; the columns go to ten
//     zero-padded LDS rows (tap-major, so that the lanes of a wave read
//     consecutive words) in two passes of ten and eight y3 rows, and each
//     logit sums its four column entries.
// Products: v_mfma_f32_16x16x32_bf16 (16x16x16 where K is 16), FP32 accumulation.
//
// What bounds it: the latency of its LDS reads and products between the six
// barriers of a strip (the products alone take 10 us at 512 sets).  Strips
// keep the LDS of a workgroup at 71 KB, so two share a CU and fill each
// other's waits, and a small batch spreads over four times the CUs; one
// workgroup a set (140 KB) had 40 barriers a set and began each with the
// loads of the linear layers.  512 sets: 37.1 + 4.7 us (strips, linear
// layers; traced in a long run of calls), before 55.9 + 4.7 us; one set: 8.3 +
// 3.7 against 25.5 + 3.7 us.
// Four waves with their weights in registers (250) read an operand row once
// for both column phases and twice over the rows; eight waves of 128
// registers, one phase each, read LDS 2.4 times as much and took 61 us where
// these, with to_bf16 in integer steps still, took 53.
constexpr int kFwdThreads = 256;                      // 4 waves
constexpr int kY1S = 64 + 8, kY2S = 32 + 8;           // bf16 per pixel: 16-byte rows, padded against bank conflicts
constexpr int kY2Bytes = 10 * 34 * kY2S * 2;          // rows 8 s - 1 .. 8 s + 8, x = -1 .. 32, the ends zero
constexpr int kColRows = 10;                          // y3 row 16 s - 1 + li in slot li % 10
constexpr int kColW = 68;                             // pixel x at entry x + 2, x = -1 .. 64, the ends zero
constexpr int kColBytes = kColRows * 16 * kColW * 4;
static_assert(6 * 18 * kY1S * 2 <= kColBytes, "the columns reuse the y1 space");
constexpr int kFwdGrid = 512;                         // two workgroups a CU

struct FwdArgs {
    const kl_c64 *ta, *tb;
    const float* P;
    Layout L;
    bf16_t *packed, *x0;
    float* logits;                                 // B x 128 x 128
    int B;
};

__device__ __forceinline__ bf16x4 relu_bf16(f32x4 d, f32x4 bias) { return round4(relu4(add4(d, bias))); }

__global__ __launch_bounds__(256) void forward_mlp_kernel(const FwdArgs a, int mlp_blocks) {
    __shared__ __align__(16) bf16_t h1s[16 * 264];
    __shared__ float us[16][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    if ((int)blockIdx.x >= mlp_blocks) {
        const int stride = (int)(gridDim.x - mlp_blocks) * 256;
        for (int e = ((int)blockIdx.x - mlp_blocks) * 256 + tid; e < kForwardPacked; e += stride)
            a.packed[e] = to_bf16(packed_weight(a.P, a.L, e));
        return;
    }
    const int b0 = ((int)blockIdx.x / 4) * 16;
    if (tid < 16) {
        const int b = min(b0 + tid, a.B - 1);
        us[tid][0] = bf16_value((float)((a.ta[b].re - 2.4) / 0.6));
        us[tid][1] = bf16_value((float)(a.ta[b].im / 0.3));
        us[tid][2] = bf16_value((float)((a.tb[b].re - 2.4) / 0.6));
        us[tid][3] = bf16_value((float)(a.tb[b].im / 0.3));
    }
    // rows o of W2^T, 16 a wave: the loads run while h1 is formed
    const int o0 = (((int)blockIdx.x % 4) * 4 + wave) * 16;
    bf16x8 w[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int k = 0; k < 8; ++k) w[ks][k] = (short)to_bf16(a.P[a.L.W2 + (ks * 32 + 8 * lq + k) * 256 + o0 + lr]);
    float w1[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w1[k] = bf16_value(a.P[a.L.W1 + k * 256 + tid]);
    const float b1 = a.P[a.L.b1 + tid];
    __syncthreads();
#pragma unroll 4
    for (int q = 0; q < 16; ++q) {
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc = fmaf(us[q][k], w1[k], acc);
        h1s[q * 264 + tid] = to_bf16(fmaxf(acc + b1, 0.f));
    }
    __syncthreads();
    f32x4 d = kZero4;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) d = mma32(w[ks], lds8(h1s + lr * 264 + ks * 32 + 8 * lq), d);
    if (b0 + lr < a.B) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int o = o0 + 4 * lq + v;   // feature c * 16 + q -> x0 pixel q, channel c
            a.x0[((size_t)(b0 + lr) * 16 + o % 16) * 16 + o / 16] = to_bf16(fmaxf(d[v] + a.P[a.L.b2 + o], 0.f));
        }
    }
}

// Strips dealt round robin over the grid: 4 a set.  Four waves, all weights
// in registers: a wave takes one output row parity of each stride-2 layer
// (and 16 of the channels, or half of the columns), so the three shifted
// operands it reads of an input row serve both column phases, and the row's
// next use, one output row on, finds them in registers.
__global__ __launch_bounds__(kFwdThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void forward_kernel(const FwdArgs a) {
    __shared__ __align__(16) unsigned char dsm[kY2Bytes + kColBytes];
    bf16_t* y2p = (bf16_t*)dsm;                                // [10][34][kY2S]
    bf16_t* y1p = (bf16_t*)(dsm + kY2Bytes);                   // [6][18][kY1S]
    float* col = (float*)(dsm + kY2Bytes);                     // [kColRows][16 taps][kColW], once y1 is consumed
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4, half = wave & 1, py = wave >> 1;

    bf16x4 w1[4][4];    // convT 1: taps (wave, kx), 16 channels each
#pragma unroll
    for (int kx = 0; kx < 4; ++kx)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) w1[kx][ct] = frag4(a.packed + kT1f, (4 * wave + kx) * 4 + ct, lane);
    bf16x8 w2[2][8];    // convT 2: both column phases, (tap, channel half); output channels 16 half ..
    bf16x8 w3[2][4];    // convT 3: both column phases, tap; columns 2 (16 half + lr) + px
#pragma unroll
    for (int px = 0; px < 2; ++px) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            w2[px][ks] = frag8(a.packed + kI2, ((2 * py + px) * 8 + ks) * 2 + half, lane);
#pragma unroll
        for (int tap = 0; tap < 4; ++tap) w3[px][tap] = frag8(a.packed + kI3, (2 * py + px) * 4 + tap, lane);
    }
    const bf16x4 w4 = frag4(a.packed + kT4f, 0, lane);
    f32x4 bias1[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) bias1[ct] = load4(a.P + a.L.c1 + 16 * ct + 4 * lq);
    const f32x4 bias2 = load4(a.P + a.L.c2 + 16 * half + 4 * lq), bias3 = load4(a.P + a.L.c3 + 4 * lq);
    const float bias4 = a.P[a.L.c4];

    if (tid < 10 * 2 * 5) {   // the ends of the y2 rows stay zero
        const int g = tid % 5, e = (tid / 5) & 1, r = tid / 10;
        ((uint4*)(y2p + (r * 34 + (e ? 33 : 0)) * kY2S))[g] = make_uint4(0, 0, 0, 0);
    }
    for (int unit = blockIdx.x; unit < 4 * a.B; unit += gridDim.x) {
        const int b = unit >> 2, s = unit & 3;
        const bf16x4 x = loadw(a.x0 + ((size_t)b * 16 + lr) * 16 + 4 * lq);
        // y1 rows 4 s - 1 .. 4 s + 4: the row beyond the grid and the ends zero
        if (tid < 6 * 2 * 9) {
            const int g = tid % 9, e = (tid / 9) & 1, r = tid / 18;
            ((uint4*)(y1p + (r * 18 + (e ? 17 : 0)) * kY1S))[g] = make_uint4(0, 0, 0, 0);
        }
        if ((s == 0 || s == 3) && tid >= 256 - 16 * 9)
            ((uint4*)(y1p + ((s ? 5 : 0) * 18 + 1) * kY1S))[tid - (256 - 16 * 9)] = make_uint4(0, 0, 0, 0);
        {
            const int i = lr >> 2, j = lr & 3, row = 4 * i + wave - (4 * s - 1);
            const bool in = row >= 0 && row < 6;
#pragma unroll
            for (int kx = 0; kx < 4; ++kx)
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
                    const bf16x4 y = relu_bf16(mma16(w1[kx][ct], x, kZero4), bias1[ct]);
                    if (in) *(bf16x4*)(y1p + (row * 18 + 4 * j + kx + 1) * kY1S + 16 * ct + 4 * lq) = y;
                }
        }
        __syncthreads();
        // y2 rows 8 s - 1 .. 8 s + 8 of this wave's parity: local rows 2 t + 1 - py, from the local
        // y1 rows t + 1 (first row tap) and t (second)
        {
            bf16x8 f[2][3][2];   // [row & 1][shift -1, 0, 1][channel half]
            auto rows = [&](int r) {
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int h = 0; h < 2; ++h) f[r & 1][dx][h] = lds8(y1p + (r * 18 + lr + dx) * kY1S + 32 * h + 8 * lq);
            };
            rows(0);
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                rows(t + 1);
                const int r = 2 * t + 1 - py, Y = 8 * s - 1 + r;
                f32x4 d[2] = {kZero4, kZero4};
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                    for (int px = 0; px < 2; ++px)
                        d[px] = mma32(w2[px][ks], f[(t + 1 - (ks >> 2)) & 1][tap_dy(px, (ks >> 1) & 1) + 1][ks & 1], d[px]);
#pragma unroll
                for (int px = 0; px < 2; ++px) {
                    bf16x4 y = relu_bf16(d[px], bias2);
                    if (Y < 0 || Y >= 32) y = bf16x4{0, 0, 0, 0};
                    *(bf16x4*)(y2p + (r * 34 + 2 * lr + px + 1) * kY2S + 16 * half + 4 * lq) = y;
                }
            }
        }
        __syncthreads();
        for (int i = tid; i < kColRows * 16 * 2; i += kFwdThreads) col[(i >> 1) * kColW + ((i & 1) ? 66 : 1)] = 0.f;
        // y3 rows li = 0 .. 9, then 10 .. 17 (row 16 s - 1 + li), and the logits they complete
        bf16x8 f[2][3];   // [row & 1][shift]
        auto rows = [&](int r) {
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) f[r & 1][dx] = lds8(y2p + (r * 34 + 16 * half + lr + dx) * kY2S + 8 * lq);
        };
        rows(0);
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int t = pass ? 5 : 0; t < (pass ? 9 : 5); ++t) {
                rows(t + 1);
                const int li = 2 * t + 1 - py, Y = 16 * s - 1 + li;
                f32x4 d[2] = {kZero4, kZero4}, c[2];
#pragma unroll
                for (int tap = 0; tap < 4; ++tap)
#pragma unroll
                    for (int px = 0; px < 2; ++px)
                        d[px] = mma32(w3[px][tap], f[(t + 1 - (tap >> 1)) & 1][tap_dy(px, tap & 1) + 1], d[px]);
#pragma unroll
                for (int px = 0; px < 2; ++px) c[px] = mma16(w4, relu_bf16(d[px], bias3), kZero4);   // taps 4 lq .. + 3
                const bool in = Y >= 0 && Y < 64;
                float* row = col + (li % kColRows) * 16 * kColW + 2 * (16 * half + lr) + 2;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    *(float2*)(row + (4 * lq + v) * kColW) = make_float2(in ? c[0][v] : 0.f, in ? c[1][v] : 0.f);
            }
            __syncthreads();
            // logit rows 32 s + 16 pass .. + 15, columns 2u and 2u + 1: X = 2u takes pixels u
            // (kx 1) and u - 1 (kx 3), X = 2u + 1 pixels u + 1 (kx 0) and u (kx 2)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int zl = 16 * pass + 4 * q + wave, Z = 32 * s + zl, u = lane;
                float e0 = 0.f, e1 = 0.f;
#pragma unroll
                for (int ra = 0; ra < 2; ++ra) {
                    // taps (ky, 0..3) of y3 row (Z >> 1) + dy; pixel x is column entry x + 2
                    const int li = (zl >> 1) + 1 + tap_dy(Z & 1, ra);
                    const float* t = col + ((li % kColRows) * 16 + 4 * tap_k(Z & 1, ra)) * kColW + u + 1;
                    e0 += t[kColW + 1] + t[3 * kColW];
                    e1 += t[2] + t[2 * kColW + 1];
                }
                *(float2*)(a.logits + ((int64_t)b * 128 + Z) * 128 + 2 * u) = make_float2(e0 + bias4, e1 + bias4);
            }
            __syncthreads();   // the next rows, or the next strip's y1, overwrite the columns
        }
    }
}

static unsigned grid_for(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(8192, (n + 255) / 256)); }

// Inference forward: linear layers and packed weights, then the strips.
static hipError_t forward_fused(const float* P, const kl_c64* ta, const kl_c64* tb, int B, float* logits,
                                const WS& w, hipStream_t s) {
    const FwdArgs f{ta, tb, P, layout(), w.packed, w.x0h, logits, B};
    const int mlp = 4 * ((B + 15) / 16);
    hipLaunchKernelGGL(forward_mlp_kernel, dim3(mlp + 112), dim3(256), 0, s, f, mlp);
    hipLaunchKernelGGL(forward_kernel, dim3(std::min(4 * B, kFwdGrid)), dim3(kFwdThreads), 0, s, f);
    return hipGetLastError();
}

}  // namespace sur
}  // namespace kl

using namespace kl;
using namespace kl::sur;

static int sur_fail(int code, const char* m) { return set_error(code, "%s", m); }

extern "C" {

size_t kl_sur_num_params(void) { return layout().total; }

size_t kl_sur_workspace_bytes(int batch) { return batch > 0 ? carve(nullptr, batch).bytes : 0; }

int kl_sur_workspace_tensor(int batch, int which, size_t* offset_bytes, size_t* n_floats) {
    if (batch <= 0 || !offset_bytes || !n_floats) return sur_fail(KL_EINVAL, "bad workspace query");
    const WS w = carve(nullptr, batch);
    const WS z = carve((void*)(uintptr_t)256, batch);   // offsets relative to a nonzero base
    const size_t b = (size_t)batch;
    const float* p = nullptr;
    size_t n = 0;
    switch (which) {
        case KL_SUR_T_U: p = z.u; n = b * 4; break;
        case KL_SUR_T_H1: p = z.h1; n = b * 256; break;
        case KL_SUR_T_H2: p = z.h2; n = b * 256; break;
        case KL_SUR_T_X0: p = z.x0; n = b * 256; break;
        case KL_SUR_T_Y1: p = z.y1; n = b * 256 * 64; break;
        case KL_SUR_T_Y2: p = z.y2; n = b * 1024 * 32; break;
        case KL_SUR_T_Y3: p = z.y3; n = b * 4096 * 16; break;
        case KL_SUR_T_LOGITS: p = z.logits; n = b * kImg * kImg; break;
        case KL_SUR_T_DLOGITS: p = z.dlogits; n = b * kImg * kImg; break;
        case KL_SUR_T_DY3: p = z.dy3; n = b * 4096 * 16; break;
        case KL_SUR_T_DY2: p = z.dy2; n = b * 1024 * 32; break;
        case KL_SUR_T_DY1: p = z.dy1; n = b * 256 * 64; break;
        case KL_SUR_T_DX0: p = z.dx0; n = b * 256; break;
        case KL_SUR_T_DH2: p = z.dh2; n = b * 256; break;
        case KL_SUR_T_DH1: p = z.dh1; n = b * 256; break;
        default: return sur_fail(KL_EINVAL, "unknown workspace tensor");
    }
    (void)w;
    *offset_bytes = (size_t)((const char*)p - (const char*)(uintptr_t)256);
    *n_floats = n;
    return KL_OK;
}

int kl_gemm_bf16(int M, int N, int K, const float* A, int64_t lda_m, int64_t lda_k, const float* B, int64_t ldb_k,
                 int64_t ldb_n, float* C, int64_t ldc, const float* bias, int relu, int accumulate, void* stream) {
    if (M < 0 || N < 0 || K < 0) return sur_fail(KL_EINVAL, "negative GEMM size");
    if (M == 0 || N == 0) return KL_OK;
    if ((K > 0 && (!A || !B)) || !C) return sur_fail(KL_EINVAL, "NULL GEMM operand");
    if (accumulate && (bias || relu)) return sur_fail(KL_EINVAL, "accumulate excludes bias and relu");
    hipError_t e = gemm(M, N, K, A, lda_m, lda_k, B, ldb_k, ldb_n, C, ldc, bias, relu, accumulate, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

int kl_sur_forward(const float* params, const kl_c64* ta, const kl_c64* tb, int batch, float* logits_out,
                   void* workspace, size_t workspace_bytes, void* stream) {
    if (batch > 512) return sur_fail(KL_EINVAL, "batch above 512");
    if (batch <= 0 || !params || !ta || !tb || !logits_out || !workspace)
        return sur_fail(KL_EINVAL, "bad surrogate forward arguments");
    if (workspace_bytes < kl_sur_workspace_bytes(batch)) return sur_fail(KL_EINVAL, "workspace too small");
    const WS w = carve(workspace, batch);
    hipError_t e = forward_fused(params, ta, tb, batch, logits_out, w, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

static Adam adam_args(float* params, float* m, float* v, int step, float lr) {
    return {params, m, v, lr, 1.f - powf(0.9f, (float)step), 1.f - powf(0.999f, (float)step)};
}

static int sur_loss_grad(const float* params, const kl_c64* ta, const kl_c64* tb, const uint8_t* targets, int batch,
                         float* grad_out, float* loss_out, const Adam& adam, void* workspace, size_t workspace_bytes,
                         void* stream) {
    if (batch > 512) return sur_fail(KL_EINVAL, "batch above 512");
    if (batch <= 0 || !params || !ta || !tb || !targets || !grad_out || !loss_out || !workspace)
        return sur_fail(KL_EINVAL, "bad surrogate gradient arguments");
    if (workspace_bytes < kl_sur_workspace_bytes(batch)) return sur_fail(KL_EINVAL, "workspace too small");
    const WS w = carve(workspace, batch);
    hipError_t e = loss_grad(params, ta, tb, targets, batch, grad_out, loss_out, adam, w, (hipStream_t)stream);
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

int kl_sur_loss_grad(const float* params, const kl_c64* ta, const kl_c64* tb, const uint8_t* targets, int batch,
                     float* grad_out, float* loss_out, void* workspace, size_t workspace_bytes, void* stream) {
    return sur_loss_grad(params, ta, tb, targets, batch, grad_out, loss_out, Adam{}, workspace, workspace_bytes, stream);
}

int kl_sur_adam(float* params, const float* grad, float* m, float* v, int step, float lr, void* stream) {
    if (!params || !grad || !m || !v || step < 1) return sur_fail(KL_EINVAL, "bad Adam arguments");
    const int64_t n = (int64_t)layout().total;
    hipLaunchKernelGGL(adam_kernel, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream,
                       adam_args(params, m, v, step, lr), grad, n);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

int kl_sur_train_step(float* params, float* m, float* v, float* grad_scratch, int step, float lr, const kl_c64* ta,
                      const kl_c64* tb, const uint8_t* targets, int batch, float* loss_out, void* workspace,
                      size_t workspace_bytes, void* stream) {
    if (!grad_scratch) return sur_fail(KL_EINVAL, "grad_scratch is NULL");
    const bool ok = m && v && step >= 1;   // otherwise the gradient is still formed, then the update refused
    int rc = sur_loss_grad(params, ta, tb, targets, batch, grad_scratch, loss_out,
                           ok ? adam_args(params, m, v, step, lr) : Adam{}, workspace, workspace_bytes, stream);
    return rc || ok ? rc : kl_sur_adam(params, grad_scratch, m, v, step, lr, stream);
}

int kl_occupancy(const uint32_t* counts, uint64_t n, uint8_t* occ_out, void* stream) {
    if (n == 0) return KL_OK;
    if (!counts || !occ_out) return sur_fail(KL_EINVAL, "NULL occupancy buffer");
    hipLaunchKernelGGL(occupancy_kernel, dim3(grid_for((int64_t)std::min<uint64_t>(n, 1ull << 40))), dim3(256), 0,
                       (hipStream_t)stream, counts, n, occ_out);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

int kl_sur_predict_occupancy(const float* logits, uint64_t n, uint8_t* occ_out, void* stream) {
    if (n == 0) return KL_OK;
    if (!logits || !occ_out) return sur_fail(KL_EINVAL, "NULL occupancy buffer");
    hipLaunchKernelGGL(predict_occupancy_kernel, dim3(grid_for((int64_t)std::min<uint64_t>(n, 1ull << 40))), dim3(256),
                       0, (hipStream_t)stream, logits, n, occ_out);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

int kl_sur_uncertainty(const float* logits, int batch, float* out, void* stream) {
    if (batch <= 0 || !logits || !out) return sur_fail(KL_EINVAL, "bad uncertainty arguments");
    hipLaunchKernelGGL(uncertainty_kernel, dim3(batch), dim3(kUncThreads), 0, (hipStream_t)stream, logits, out);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

int kl_iou(const float* logits, const uint8_t* pred_occ, const uint8_t* target_occ, int batch, float* iou_out,
           void* stream) {
    if (batch <= 0 || (!logits && !pred_occ) || !target_occ || !iou_out)
        return sur_fail(KL_EINVAL, "bad IoU arguments");
    hipLaunchKernelGGL(iou_kernel, dim3(batch), dim3(256), 0, (hipStream_t)stream, logits, pred_occ, target_occ,
                       iou_out);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? KL_OK : sur_fail(KL_EDEVICE, hipGetErrorString(e));
}

}  // extern "C"
