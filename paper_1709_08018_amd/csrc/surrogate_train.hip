// surrogate_train.hip -- one training step's loss and gradient for the
// occupancy surrogate (include/kl_surrogate.h).
//
// Every product runs on the matrix cores with its operands rounded to
// bfloat16 on their way into LDS or registers, and accumulates in FP32; the
// layers' FP32 inputs, outputs and gradients stay in the workspace
// (kl_sur_workspace_tensor), NHWC.  No column matrix is formed: a transposed
// convolution gathers its input pixels from LDS, phase by phase, and the
// backward products read the output's gradient from LDS planes (one per
// channel), where the four kx taps of a row are four consecutive entries.
//
// What bounds it: the FP32 tensors a step leaves in the workspace (1.1 MB a
// set, written once and read once or twice, 143 MB written at 128 sets) and
// the latency of eight dependent launches; the products are 14 GFLOP.  A step
// of 128 sets takes 113-120 us, of 8 sets 59 us; with column matrices in memory
// (a GEMM into them or out of them per layer, 560 MB of columns) 128 sets took
// 1371 us, with weights read in the parameters' own order 159 us.
//
// Sums that feed another rounding keep one fixed order (below, per kernel):
// each tap's product over the input channels on its own, 16 channels a
// matrix instruction, then the taps in ascending (ky, kx) and the bias.
// Weight and bias gradients are summed per workgroup and then over the
// workgroups in a fixed order: no atomics, so a step repeats bit for bit.
#include <algorithm>

#include "surrogate.hpp"

namespace kl {
namespace sur {

namespace {

// Keeps a loaded value in its registers from here on: the compiler would
// otherwise move the load down to its use, inside the chain of products, where
// every group of four cost a microsecond of latency.
__device__ __forceinline__ void hold(bf16x4& v) { asm volatile("" : "+v"(v)); }

// two consecutive LDS dwords as four bfloat16 values
__device__ __forceinline__ bf16x4 lds_taps(const uint32_t* p) {
    const uint2 u = {p[0], p[1]};
    return __builtin_bit_cast(bf16x4, u);
}
// every second bfloat16 value of four consecutive LDS dwords: the low halves
// (sel 0x05040100) or the high ones (0x07060302)
__device__ __forceinline__ bf16x4 lds_stride2(const uint32_t* p, uint32_t sel) {
    const uint2 u = {__builtin_amdgcn_perm(p[1], p[0], sel), __builtin_amdgcn_perm(p[3], p[2], sel)};
    return __builtin_bit_cast(bf16x4, u);
}

// g where the activation y is positive, else 0
__device__ __forceinline__ f32x4 mask4(f32x4 g, f32x4 y) {
    f32x4 r;
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = y[v] > 0.f ? g[v] : 0.f;
    return r;
}
// A product leaves lane l with four channels (4 (l / 16) ..) of pixel l % 16:
// in memory order, lane l holds the l-th 16 bytes of the sixteen pixels'
// channels.  A store in the first order is 64 requests, in the second sixteen,
// for four shuffles.
__device__ __forceinline__ f32x4 to_memory(f32x4 v, int lane) {
    const int src = (lane & 3) * 16 + (lane >> 2);
    return f32x4{__shfl(v[0], src, 64), __shfl(v[1], src, 64), __shfl(v[2], src, 64), __shfl(v[3], src, 64)};
}
// sum over the 16 lanes that share lane / 16
__device__ __forceinline__ float sum16(float x) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// sum over the 16 lanes that share lane % 4 (memory order)
__device__ __forceinline__ float sum_rows(float x) {
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// log(1 + e^-|z|) from x = e^-z, as 2 atanh(s) with s = e^-|z| / (2 + e^-|z|),
// the atanh by its power series to s^15 (s <= 1/3: truncated below 2e-9 of
// its value).  x = infinity, or below FP32's range, gives 0.
__device__ __forceinline__ float softplus_abs(float z, float x) {
    const float n = z >= 0.f ? x : 1.f, d = z >= 0.f ? 2.f + x : 1.f + 2.f * x, s = n / d, y = s * s;
    float c = 1.f / 15.f;
    c = fmaf(c, y, 1.f / 13.f);
    c = fmaf(c, y, 1.f / 11.f);
    c = fmaf(c, y, 1.f / 9.f);
    c = fmaf(c, y, 1.f / 7.f);
    c = fmaf(c, y, 1.f / 5.f);
    c = fmaf(c, y, 1.f / 3.f);
    return fmaf(2.f * s, c * y, 2.f * s);
}

struct TrainArgs {
    const float* P;                  // parameters
    const kl_c64 *ta, *tb;
    const uint8_t* targets;
    WS w;
    Layout L;
    int B;
    int chunk3, chunk2;              // output channels summed in one chain in dy2 and dy1 (sum_chunk)
};

// The input gradients of the second and third layers sum K = Co * 16 terms
// in chains that start anew every `chunk` output channels; the chains' sums
// are then added in order.  Batches with fewer than 512 tiles of 64 x 64
// results take 1024 / tiles chains, at least eight channels each (the rule
// that gemm() splits K by), larger ones a single chain: the order is part of
// what a batch's gradient is, bit for bit.
int sum_chunk(int rows, int Co) {
    const int tiles = (rows + 63) / 64;
    if (tiles >= 512) return Co;
    const int split = std::min(Co / 8, std::max(1, 1024 / tiles));
    return ((Co + split - 1) / split + 3) / 4 * 4;
}

// Planes of one gradient tensor in LDS: `rows` rows from y0 on of the W x W x C
// tensor d (NHWC), channels c0 .. c0 + 4 CG - 1, one bfloat16 plane a channel
// (RW dwords a row, RP a plane), entry X + 1 of a row, X = -1 .. W, zero
// outside.  A task is a pixel pair by four channels; every load is issued
// before the first is used.
template <int THREADS, int W, int C, int CG, int ROWS, int RW, int RP>
__device__ __forceinline__ void load_planes(const float* __restrict__ d, int y0, int c0, uint32_t* pl, int tid) {
    constexpr int PAIRS = W / 2 + 1, TASKS = ROWS * PAIRS * CG, N = (TASKS + THREADS - 1) / THREADS;
    constexpr int STEP = THREADS / CG;   // pairs from a thread's task to its next
    static_assert(THREADS % CG == 0, "a thread keeps its channels");
    const int cg = tid % CG, j0 = (tid / CG) % PAIRS, r0 = tid / (CG * PAIRS);
    f32x4 v[N][2];
    int j = j0, r = r0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int y = y0 + r;
        const float* p = d + (y * W + 2 * j) * C + c0 + 4 * cg;
        const bool in = y >= 0 && y < W && (q < N - 1 || r < ROWS);
        v[q][0] = in && j > 0 ? load4(p - C) : kZero4;
        v[q][1] = in && j < W / 2 ? load4(p) : kZero4;
        j += STEP % PAIRS;
        r += STEP / PAIRS + (j >= PAIRS ? 1 : 0);
        j -= j >= PAIRS ? PAIRS : 0;
    }
    j = j0;
    r = r0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        if (q < N - 1 || r < ROWS) {
            uint32_t* t = pl + 4 * cg * RP + r * RW + j;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e * RP] = pack2(v[q][0][e], v[q][1][e]);
        }
        j += STEP % PAIRS;
        r += STEP / PAIRS + (j >= PAIRS ? 1 : 0);
        j -= j >= PAIRS ? PAIRS : 0;
    }
}

// N pixels of an activation (C channels, NHWC, from x on) transposed into LDS as
// bfloat16: channel c's pixels at t[c * (TW dwords)], two a dword.
template <int THREADS, int N, int C, int TW>
__device__ __forceinline__ void load_transposed(const float* __restrict__ x, uint32_t* t, int tid) {
    constexpr int CG = C / 4, TASKS = N / 2 * CG, Q = TASKS / THREADS;
    static_assert(TASKS % THREADS == 0, "whole rounds");
    f32x4 v[Q][2];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int i = tid + THREADS * q, cg = i % CG, j = i / CG;
        const float* p = x + (2 * j) * C + 4 * cg;
        v[q][0] = load4(p);
        v[q][1] = load4(p + C);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int i = tid + THREADS * q, cg = i % CG, j = i / CG;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[(4 * cg + e) * TW + j] = pack2(v[q][0][e], v[q][1][e]);
    }
}

// ------------------------------------------------------------------ linear layers and weight packing
// Blocks below mlp_blocks: 16 sets and 64 outputs of the second linear layer
// (each block forms the first layer of its sets, 16 instructions).  The
// others round the weights to bfloat16 in the order the products read them.
__global__ __launch_bounds__(256) void prologue_kernel(const TrainArgs a, int mlp_blocks) {
    __shared__ __align__(16) bf16_t h1s[16 * 264];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= mlp_blocks) {
        const int stride = (int)(gridDim.x - mlp_blocks) * 256;
        constexpr int kSkip = kForwardPacked - kI2;   // the inference path's fragments
        for (int i = ((int)blockIdx.x - mlp_blocks) * 256 + tid; i < kTrainPacked - kSkip; i += stride) {
            const int e = i < kI2 ? i : i + kSkip;
            a.w.packed[e] = to_bf16(packed_weight(a.P, a.L, e));
        }
        return;
    }
    const int b0 = ((int)blockIdx.x / 4) * 16, nb = (int)blockIdx.x % 4;
    const float *W1 = a.P + a.L.W1, *b1 = a.P + a.L.b1, *W2 = a.P + a.L.W2, *b2 = a.P + a.L.b2;
    // features of set b0 + lr, in lanes 0..15 of each wave (the four k values of the product)
    f32x4 u = kZero4;
    if (lq == 0 && b0 + lr < a.B) {
        const int b = b0 + lr;
        u[0] = (float)((a.ta[b].re - 2.4) / 0.6);
        u[1] = (float)(a.ta[b].im / 0.3);
        u[2] = (float)((a.tb[b].re - 2.4) / 0.6);
        u[3] = (float)(a.tb[b].im / 0.3);
        if (nb == 0 && wave == 0) store4(a.w.u + 4 * b, u);
    }
    const bf16x4 ua = round4(u);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int n = (4 * wave + t) * 16 + lr;
        f32x4 wv = kZero4;
        if (lq == 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) wv[k] = W1[k * 256 + n];
        f32x4 d = mma16(ua, round4(wv), kZero4);
        const float bias = b1[n];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float h = fmaxf(d[v] + bias, 0.f);
            h1s[(4 * lq + v) * 264 + n] = to_bf16(h);
            if (nb == wave && b0 + 4 * lq + v < a.B) a.w.h1[(size_t)(b0 + 4 * lq + v) * 256 + n] = h;
        }
    }
    __syncthreads();
    const int n = (4 * nb + wave) * 16 + lr;   // h2 feature c * 16 + q -> x0 pixel q, channel c
    f32x4 d = kZero4;
#pragma unroll 4
    for (int k0 = 0; k0 < 256; k0 += 16) {
        f32x4 wv;
#pragma unroll
        for (int k = 0; k < 4; ++k) wv[k] = W2[(k0 + 4 * lq + k) * 256 + n];
        d = mma16(lds4(h1s + lr * 264 + k0 + 4 * lq), round4(wv), d);
    }
    const float bias = b2[n];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int b = b0 + 4 * lq + v;
        if (b < a.B) {
            const float h = fmaxf(d[v] + bias, 0.f);
            a.w.h2[(size_t)b * 256 + n] = h;
            a.w.x0[((size_t)b * 16 + n % 16) * 16 + n / 16] = h;
        }
    }
}

// ------------------------------------------------------------------ forward: first two transposed convolutions
// One workgroup per (set, 4 rows m of y1): y1 rows 4 s - 1 .. 4 s + 4 in LDS
// (the neighbours' rows formed again: 64 matrix instructions), then y2 rows
// 8 s .. 8 s + 7, one output phase a wave.
constexpr int kY1P = 64 + 8, kY2P = 32 + 8;   // bf16 per pixel in LDS, padded against bank conflicts

__global__ __launch_bounds__(256) void conv12_kernel(const TrainArgs a) {
    __shared__ __align__(16) bf16_t y1s[6 * 18 * kY1P];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = (int)blockIdx.x >> 2, s = (int)blockIdx.x & 3;
    const bf16_t* T = a.w.packed;
    for (int i = tid; i < 6 * 18 * kY1P / 8; i += 256) ((uint4*)y1s)[i] = make_uint4(0, 0, 0, 0);
    // every weight and bias is asked for before the first is used
    bf16x4 w1[4][4];
    f32x4 bias1[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        bias1[ct] = load4(a.P + a.L.c1 + 16 * ct + 4 * lq);
#pragma unroll
        for (int kx = 0; kx < 4; ++kx) w1[ct][kx] = frag4(T + kT1f, (4 * wave + kx) * 4 + ct, lane);
    }
    const bf16x4 x = round4(load4(a.w.x0 + ((size_t)b * 16 + lr) * 16 + 4 * lq));
    const int py = wave >> 1, px = wave & 1;
    bf16x4 w[2][4][4];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int tap = 0; tap < 4; ++tap)
#pragma unroll
            for (int kc = 0; kc < 4; ++kc)
                w[ct][tap][kc] = frag4(T + kT2f, ((wave * 4 + tap) * 2 + ct) * 4 + kc, lane);
    const f32x4 bias20 = load4(a.P + a.L.c2 + 4 * lq), bias21 = load4(a.P + a.L.c2 + 16 + 4 * lq);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        hold(w1[i / 4][i % 4]);
        hold(w[0][i / 4][i % 4]);
        hold(w[1][i / 4][i % 4]);
    }
    __syncthreads();
    {
        const int i = lr >> 2, j = lr & 3, ky = wave;   // input pixel (i, j); output row 4 i + ky
        const int row = 4 * i + ky - (4 * s - 1);
        const bool in = row >= 0 && row < 6, own = i == s;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const f32x4 bias = bias1[ct];
#pragma unroll
            for (int kx = 0; kx < 4; ++kx) {
                const f32x4 d = mma16(w1[ct][kx], x, kZero4);
                const f32x4 y = relu4(add4(d, bias));
                if (in) *(bf16x4*)(y1s + (row * 18 + 4 * j + kx + 1) * kY1P + 16 * ct + 4 * lq) = round4(y);
                if (own) store4(a.w.y1 + (((size_t)b * 16 + 4 * i + ky) * 16 + 4 * j + kx) * 64 + 16 * ct + 4 * lq, y);
            }
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int mi = 0; mi < 4; ++mi) {
        f32x4 s0 = kZero4, s1 = kZero4;
#pragma unroll
        for (int tap = 0; tap < 4; ++tap) {
            const bf16_t* p = y1s + ((mi + 1 + tap_dy(py, tap >> 1)) * 18 + lr + tap_dy(px, tap & 1) + 1) * kY1P + 4 * lq;
            f32x4 d0 = kZero4, d1 = kZero4;
#pragma unroll
            for (int kc = 0; kc < 4; ++kc) {
                const bf16x4 v = lds4(p + 16 * kc);
                d0 = mma16(w[0][tap][kc], v, d0);
                d1 = mma16(w[1][tap][kc], v, d1);
            }
            s0 = add4(s0, d0);
            s1 = add4(s1, d1);
        }
        float* y = a.w.y2 + (((size_t)b * 32 + 2 * (4 * s + mi) + py) * 32 + 2 * (lane >> 2) + px) * 32 + 4 * (lane & 3);
        store4(y, to_memory(relu4(add4(s0, bias20)), lane));
        store4(y + 16, to_memory(relu4(add4(s1, bias21)), lane));
    }
}

// ------------------------------------------------------------------ last two layers, forward and backward
// One workgroup per (set, 8 rows of y3): y3 rows 8 s - 1 .. 8 s + 8, from
// them the columns of the last layer, logit rows 16 s - 1 .. 16 s + 16 and
// their loss gradient (bfloat16, in LDS), and from those the strip's own
// rows of dy3 and its share of the gradients of K4 and of the biases.  The
// rows beyond the strip are formed again, so that y3 and the loss gradient
// are not read back from memory: 10 / 8 of the strip's products against
// 42 MB read at 128 sets.
constexpr int kDlW = 132;                     // loss gradient row: entry X + 1, X = -1 .. 128
constexpr int kColW = 66;                     // column row: entry x + 1, x = -1 .. 64
constexpr int kY3T = 8 * 64 + 8;              // y3 of one channel: entry row * 64 + x
constexpr int kStripBytes = 6 * 34 * kY2P * 2;
static_assert(18 * kDlW * 2 <= kStripBytes, "the loss gradient reuses the y2 rows' space");

__global__ __launch_bounds__(512) void conv34_kernel(const TrainArgs a) {
    __shared__ __align__(16) unsigned char lds[kStripBytes + 10 * 16 * kColW * 4];
    bf16_t* y2s = (bf16_t*)lds;                              // [6][34][kY2P]
    bf16_t* dl = (bf16_t*)lds;                               // [18][kDlW], once y2 is consumed
    float* col = (float*)(lds + kStripBytes);                // [10][16 taps][kColW]
    bf16_t* y3t = (bf16_t*)(lds + kStripBytes);              // [16][kY3T], once the columns are consumed
    float* red = (float*)(lds + kStripBytes + 16 * kY3T * 2);   // [8][256] and [8][32]
    static_assert(16 * kY3T * 2 + (8 * 256 + 8 * 32) * 4 <= 10 * 16 * kColW * 4, "scratch in the columns' space");
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = (int)blockIdx.x >> 3, s = (int)blockIdx.x & 7;
    const bf16_t* T = a.w.packed;

    // y2 rows 4 s - 1 .. 4 s + 4, zero outside
    f32x4 y2v[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int i = tid + 512 * q, g = i & 7, x = (i >> 3) & 31, y = 4 * s - 1 + (i >> 8);
        y2v[q] = kZero4;
        if (y >= 0 && y < 32) y2v[q] = load4(a.w.y2 + (((size_t)b * 32 + y) * 32 + x) * 32 + 4 * g);
    }
    if (tid < 6 * 2 * 8) {
        const int g = tid & 7, e = (tid >> 3) & 1, r = tid >> 4;
        *(bf16x4*)(y2s + (r * 34 + (e ? 33 : 0)) * kY2P + 4 * g) = bf16x4{0, 0, 0, 0};
    }
    if (tid < 320) col[(tid >> 1) * kColW + ((tid & 1) ? kColW - 1 : 0)] = 0.f;
    const int px = wave & 1, h = (wave >> 1) & 1, py = wave >> 2, x = 2 * (16 * h + lr) + px;
    const int xm = 2 * (16 * h + (lane >> 2)) + px;   // in memory order
    bf16x4 w3[4][2];
#pragma unroll
    for (int tap = 0; tap < 4; ++tap)
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
            w3[tap][kc] = frag4(T + kT3f, ((py * 2 + px) * 4 + tap) * 2 + kc, lane);
    const bf16x4 w4f = frag4(T + kT4f, 0, lane), w4b = frag4(T + kT4b, 0, lane);
    const f32x4 bias3 = load4(a.P + a.L.c3 + 4 * lq);
    const float bias4 = a.P[a.L.c4];
    uint8_t tgt[3][2] = {};   // the targets of this thread's pixels (the logits' loop below)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int i = tid + 512 * q, Z = 16 * s - 1 + (i >> 6);
        if (i < 18 * 64 && Z >= 0 && Z < kImg) {
            const uint8_t* t = a.targets + ((size_t)b * kImg + Z) * kImg + 2 * (i & 63);
            tgt[q][0] = t[0];
            tgt[q][1] = t[1];
        }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int i = tid + 512 * q, g = i & 7, x = (i >> 3) & 31, r = i >> 8;
        *(bf16x4*)(y2s + (r * 34 + x + 1) * kY2P + 4 * g) = round4(y2v[q]);
    }
    __syncthreads();

    // y3 rows of this wave's parity: local rows li = 2 t + 1 - py (row 8 s - 1 + li)
    f32x4 y3[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        const int li = 2 * t + 1 - py, Y = 8 * s - 1 + li;
        const int m = py ? t - 1 : t;   // Y >> 1, relative to 4 s
        f32x4 sum = kZero4;
#pragma unroll
        for (int tap = 0; tap < 4; ++tap) {
            const bf16_t* p = y2s + ((m + 1 + tap_dy(py, tap >> 1)) * 34 + 16 * h + lr + tap_dy(px, tap & 1) + 1) * kY2P + 4 * lq;
            sum = add4(sum, mma16(w3[tap][1], lds4(p + 16), mma16(w3[tap][0], lds4(p), kZero4)));
        }
        y3[t] = relu4(add4(sum, bias3));
        const bool in = Y >= 0 && Y < 64;
        const f32x4 c = mma16(w4f, round4(y3[t]), kZero4);   // taps 4 lq .. + 3 of pixel x
#pragma unroll
        for (int v = 0; v < 4; ++v) col[(li * 16 + 4 * lq + v) * kColW + x + 1] = in ? c[v] : 0.f;
        if (li >= 1 && li <= 8) store4(a.w.y3 + (((size_t)b * 64 + Y) * 64 + xm) * 16 + 4 * (lane & 3), to_memory(y3[t], lane));
    }
    __syncthreads();

    // logits, their loss and its gradient: row 16 s - 1 + zr, columns 2 u and 2 u + 1
    const float inv = 1.0f / (float)((int64_t)a.B * kImg * kImg);
    float loss = 0.f, dsum = 0.f;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int i = tid + 512 * q;
        if (i >= 18 * 64) break;
        const int zr = i >> 6, u = i & 63, Z = 16 * s - 1 + zr;
        float d0 = 0.f, d1 = 0.f;
        if (Z >= 0 && Z < kImg) {
            float e0 = 0.f, e1 = 0.f;
#pragma unroll
            for (int ra = 0; ra < 2; ++ra) {
                // taps (ky, 0..3) of y3 row (Z >> 1) + dy
                const float* t = col + (((Z >> 1) + tap_dy(Z & 1, ra) - (8 * s - 1)) * 16 + 4 * tap_k(Z & 1, ra)) * kColW + u;
                e0 += t[kColW + 1];
                e0 += t[3 * kColW];
                e1 += t[2];
                e1 += t[2 * kColW + 1];
            }
            e0 += bias4;
            e1 += bias4;
            const size_t at = ((size_t)b * kImg + Z) * kImg + 2 * u;
            const float t0 = tgt[q][0] ? 1.f : 0.f, t1 = tgt[q][1] ? 1.f : 0.f;
            const float x0 = expf(-e0), x1 = expf(-e1);
            d0 = (1.f / (1.f + x0) - t0) * inv;
            d1 = (1.f / (1.f + x1) - t1) * inv;
            if (zr >= 1 && zr <= 16) {
                loss += fmaxf(e0, 0.f) - e0 * t0 + softplus_abs(e0, x0);
                loss += fmaxf(e1, 0.f) - e1 * t1 + softplus_abs(e1, x1);
                dsum += d0;
                dsum += d1;
                *(float2*)(a.w.logits + at) = make_float2(e0, e1);
                *(float2*)(a.w.dlogits + at) = make_float2(d0, d1);
            }
        }
        dl[zr * kDlW + 2 * u + 1] = to_bf16(d0);
        dl[zr * kDlW + 2 * u + 2] = to_bf16(d1);
        if (u == 0) {
            dl[zr * kDlW] = 0;
            dl[zr * kDlW + kDlW - 3] = dl[zr * kDlW + kDlW - 2] = dl[zr * kDlW + kDlW - 1] = 0;
        }
    }
    __syncthreads();

    // dy3 of the strip's rows: the 16 taps of each pixel are the product's k
    const uint32_t* dlw = (const uint32_t*)dl;
    f32x4 bsum = kZero4;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        const int li = 2 * t + 1 - py;
        if (li < 1 || li > 8) continue;
        const int r = li - 1;   // row in the strip; dlogits rows 2 r + ky
        const f32x4 d = mask4(mma16(w4b, lds_taps(dlw + (2 * r + lq) * (kDlW / 2) + x), kZero4), y3[t]);
        store4(a.w.dy3 + (((size_t)b * 64 + 8 * s + r) * 64 + xm) * 16 + 4 * (lane & 3), to_memory(d, lane));
        bsum = add4(bsum, d);
#pragma unroll
        for (int v = 0; v < 4; ++v) y3t[(4 * lq + v) * kY3T + r * 64 + x] = to_bf16(y3[t][v]);
    }
    __syncthreads();

    // K4 gradient: rows channels, columns taps, k = the pixels of row `wave`, 16 at a time
    {
        const int ky = lr >> 2, kx = lr & 3;
        const uint32_t sel = (kx & 1) ? 0x07060302u : 0x05040100u;
        f32x4 g = kZero4;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            g = mma16(lds4(y3t + lr * kY3T + wave * 64 + 16 * c + 4 * lq),
                      lds_stride2(dlw + (2 * wave + ky) * (kDlW / 2) + 16 * c + 4 * lq + (kx >> 1), sel), g);
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave * 256 + (4 * lq + v) * 16 + lr] = g[v];
        float* rb = red + 8 * 256 + wave * 32;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float sv = sum16(bsum[v]);
            if (lr == 0) rb[2 + 4 * lq + v] = sv;
        }
        for (int o = 32; o > 0; o >>= 1) {
            loss += __shfl_xor(loss, o, 64);
            dsum += __shfl_xor(dsum, o, 64);
        }
        if (lane == 0) {
            rb[0] = loss;
            rb[1] = dsum;
        }
    }
    __syncthreads();
    float* part = a.w.p34 + (size_t)blockIdx.x * kPart34;
    if (tid < 256) {
        float v = 0.f;
        for (int q = 0; q < 8; ++q) v += red[q * 256 + tid];
        part[32 + tid] = v;
    } else if (tid < 256 + 18) {
        float v = 0.f;
        for (int q = 0; q < 8; ++q) v += red[8 * 256 + q * 32 + tid - 256];
        part[tid - 256] = v;
    }
}

// ------------------------------------------------------------------ backward of the third layer
// Units of (set, 8 rows of y2), dealt round robin: dy3 rows 16 s' - 1 .. + 17
// as one bfloat16 plane per channel, and y2 transposed, both in LDS.  dy2
// (masked) takes the 16 taps of one channel per matrix instruction, weights
// read four channels ahead; the K3 gradient stays in registers over a
// workgroup's units.  Bound by memory (70 MB at 128 sets) and its latency,
// hence two workgroups a CU, whose 128 registers cost 20 bytes of scratch a
// lane: 24.8 us, 28.3 us with one (188 registers, none), 39 us with all weights
// held in registers (172-264 bytes of scratch).
constexpr int kD3W = 34;                      // dwords of a dy3 plane row: entry X + 1, X = -1 .. 66
constexpr int kD3P = 18 * kD3W;               // dwords of a plane
constexpr int kY2T = 256 + 8;

__global__ __launch_bounds__(512, 4) void back3_kernel(const TrainArgs a) {
    __shared__ __align__(16) uint32_t pl[16 * kD3P];
    __shared__ __align__(16) bf16_t y2t[32 * kY2T];
    __shared__ float red[8 * 32];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bf16_t* T = a.w.packed + kT3b;
    f32x4 g[2][2] = {{kZero4, kZero4}, {kZero4, kZero4}};   // [channel o - 2 wave][input channel tile]
    f32x4 bsum[2] = {kZero4, kZero4};
    for (int unit = blockIdx.x; unit < 4 * a.B; unit += gridDim.x) {
        const int b = unit >> 2, s = unit & 3;
        int u0 = threadIdx.x;   // opaque, so that no address is kept over the units: 128 registers, two workgroups a CU
        asm volatile("" : "+v"(u0));
        const int tid = u0, lane = tid & 63, lr = lane & 15, lq = lane >> 4, ky = lr >> 2, kx = lr & 3;
        const uint32_t sel = (kx & 1) ? 0x07060302u : 0x05040100u;
        load_planes<512, 64, 16, 4, 18, kD3W, kD3P>(a.w.dy3 + (size_t)b * 4096 * 16, 16 * s - 1, 0, pl, tid);
        __builtin_amdgcn_sched_barrier(0);
        load_transposed<512, 256, 32, kY2T / 2>(a.w.y2 + ((size_t)b * 1024 + 256 * s) * 32, (uint32_t*)y2t, tid);
        __builtin_amdgcn_sched_barrier(0);
        bf16x4 w[4][2];   // four channels ahead
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) w[u][ct] = frag4(T, ct * 16 + u, lane);
        __syncthreads();
        f32x4 y2v[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
                y2v[t][ct] = load4(a.w.y2 + (((size_t)b * 32 + 8 * s + wave) * 32 + 16 * t + (lane >> 2)) * 32 + 16 * ct + 4 * (lane & 3));
        // dy2 row 8 s + wave: two tiles of 16 pixels by two of 16 channels
        f32x4 d[2][2] = {{kZero4, kZero4}, {kZero4, kZero4}}, done[2][2] = {{kZero4, kZero4}, {kZero4, kZero4}};
#pragma unroll 1
        for (int o0 = 0; o0 < 16; o0 += 4) {
            if (o0 == a.chunk3) {   // eight, or all sixteen
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) {
                        done[t][ct] = d[t][ct];
                        d[t][ct] = kZero4;
                    }
            }
            const uint32_t* p = pl + o0 * kD3P + (2 * wave + lq) * kD3W + lr;
            const int next = o0 < 12 ? o0 + 4 : 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bf16x4 v0 = lds_taps(p + u * kD3P), v1 = lds_taps(p + u * kD3P + 16);
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) {
                    d[0][ct] = mma16(w[u][ct], v0, d[0][ct]);
                    d[1][ct] = mma16(w[u][ct], v1, d[1][ct]);
                    w[u][ct] = frag4(T, ct * 16 + next + u, lane);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                const size_t at = (((size_t)b * 32 + 8 * s + wave) * 32 + 16 * t + (lane >> 2)) * 32 + 16 * ct + 4 * (lane & 3);
                const f32x4 m = mask4(to_memory(add4(done[t][ct], d[t][ct]), lane), y2v[t][ct]);
                store4(a.w.dy2 + at, m);
                bsum[ct] = add4(bsum[ct], m);
            }
        // K3 gradient of the channels 2 wave and 2 wave + 1: columns taps, k = 16 pixels of a row
#pragma unroll 2
        for (int c = 0; c < 16; ++c) {
            const bf16x4 x0 = lds4(y2t + lr * kY2T + 16 * c + 4 * lq), x1 = lds4(y2t + (16 + lr) * kY2T + 16 * c + 4 * lq);
            const uint32_t* p = pl + 2 * wave * kD3P + (2 * (c >> 1) + ky) * kD3W + 16 * (c & 1) + 4 * lq + (kx >> 1);
#pragma unroll
            for (int oi = 0; oi < 2; ++oi) {
                const bf16x4 v = lds_stride2(p + oi * kD3P, sel);
                g[oi][0] = mma16(x0, v, g[oi][0]);
                g[oi][1] = mma16(x1, v, g[oi][1]);
            }
        }
        __syncthreads();
    }
    float* part = a.w.p3 + (size_t)blockIdx.x * kPart3;
#pragma unroll
    for (int oi = 0; oi < 2; ++oi)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                part[(16 * ct + 4 * lq + v) * 256 + (2 * wave + oi) * 16 + lr] = g[oi][ct][v];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float sv = sum_rows(bsum[ct][v]);
            if (lane < 4) red[wave * 32 + 16 * ct + 4 * lane + v] = sv;
        }
    __syncthreads();
    if (tid < 32) {
        float v = 0.f;
        for (int q = 0; q < 8; ++q) v += red[q * 32 + tid];
        part[32 * 256 + tid] = v;
    }
}

// ------------------------------------------------------------------ backward of the second layer
// dy1 of one (set, 8 rows of y1) a workgroup: dy2 rows 16 s - 1 .. 16 s + 16
// as one bfloat16 plane per channel; a wave takes 16 of the 64 channels and
// four rows of 16 pixels, its weights read four channels ahead (with all 32
// held, 141 registers and one workgroup a CU: 52 us at 512 sets, 39 us so).
constexpr int kD2W = 18;                      // dwords of a dy2 plane row: entry X + 1, X = -1 .. 34

__device__ __forceinline__ void dy1_strip(const TrainArgs& a, uint32_t* pl, float* red, int blk) {
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blk >> 1, s = blk & 1;
    const int ct = wave & 3, r0 = 4 * (wave >> 2);
    bf16x4 w[4];   // four channels ahead
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = frag4(a.w.packed + kT2b, ct * 32 + u, lane);
    f32x4 y1v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) y1v[r] = load4(a.w.y1 + (((size_t)b * 16 + 8 * s + r0 + r) * 16 + (lane >> 2)) * 64 + 16 * ct + 4 * (lane & 3));
    load_planes<512, 32, 32, 8, 18, kD2W, 18 * kD2W>(a.w.dy2 + (size_t)b * 1024 * 32, 16 * s - 1, 0, pl, tid);
    __syncthreads();
    f32x4 d[4] = {kZero4, kZero4, kZero4, kZero4}, done[4] = {kZero4, kZero4, kZero4, kZero4};
    int chain = a.chunk2;   // a multiple of four
#pragma unroll 1
    for (int o0 = 0; o0 < 32; o0 += 4) {
        if (o0 == chain) {
            chain += a.chunk2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                done[r] = add4(done[r], d[r]);
                d[r] = kZero4;
            }
        }
        const uint32_t* p = pl + (o0 * 18 + 2 * r0 + lq) * kD2W + lr;
        const int next = ct * 32 + (o0 < 28 ? o0 + 4 : 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int r = 0; r < 4; ++r) d[r] = mma16(w[u], lds_taps(p + (u * 18 + 2 * r) * kD2W), d[r]);
            w[u] = frag4(a.w.packed + kT2b, next + u, lane);
        }
    }
    f32x4 bsum = kZero4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const size_t at = (((size_t)b * 16 + 8 * s + r0 + r) * 16 + (lane >> 2)) * 64 + 16 * ct + 4 * (lane & 3);
        const f32x4 m = mask4(to_memory(add4(done[r], d[r]), lane), y1v[r]);
        store4(a.w.dy1 + at, m);
        bsum = add4(bsum, m);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float sv = sum_rows(bsum[v]);
        if (lane < 4) red[(wave >> 2) * 64 + 16 * ct + 4 * lane + v] = sv;
    }
    __syncthreads();
    if (tid < 64) a.w.pc1[(size_t)blk * 64 + tid] = red[tid] + red[64 + tid];
}

// K2 gradient: a workgroup takes 8 of the 32 output channels (from o0 on)
// over every `parts`-th set, one channel a wave, all 64 input channels.
constexpr int kY1T = 256 + 8;

__device__ __forceinline__ void k2_gradient(const TrainArgs& a, uint32_t* pl, bf16_t* y1t, int part0, int parts, int o0) {
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ky = lr >> 2, kx = lr & 3;
    const uint32_t sel = (kx & 1) ? 0x07060302u : 0x05040100u;
    f32x4 g[4] = {kZero4, kZero4, kZero4, kZero4};
    for (int b = part0; b < a.B; b += parts) {
        load_planes<512, 32, 32, 2, 34, kD2W, 34 * kD2W>(a.w.dy2 + (size_t)b * 1024 * 32, -1, o0, pl, tid);
        load_transposed<512, 256, 64, kY1T / 2>(a.w.y1 + (size_t)b * 256 * 64, (uint32_t*)y1t, tid);
        __syncthreads();
#pragma unroll 4
        for (int c = 0; c < 16; ++c) {   // row c of y1
            const bf16x4 v = lds_stride2(pl + (wave * 34 + 2 * c + ky) * kD2W + 4 * lq + (kx >> 1), sel);
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) g[ct] = mma16(lds4(y1t + (16 * ct + lr) * kY1T + 16 * c + 4 * lq), v, g[ct]);
        }
        __syncthreads();
    }
    float* part = a.w.p2 + (size_t)part0 * kPart2;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[(16 * ct + 4 * lq + v) * 512 + (o0 + wave) * 16 + lr] = g[ct][v];
}

// Both need dy2 alone, so one launch does them: 4 * parts workgroups the
// gradient (the longer ones first), then 2 B dy1, two a CU, so that one's
// loads run under the other's products: 21.0 us at 128 sets, 26.4 us as two
// launches.
__global__ __launch_bounds__(512) void back2_kernel(const TrainArgs a, int parts) {
    __shared__ __align__(16) char lds[8 * 34 * kD2W * 4 + 64 * kY1T * 2];
    static_assert(32 * 18 * kD2W * 4 + 2 * 64 * 4 <= sizeof(lds), "dy1's planes in the same space");
    uint32_t* pl = (uint32_t*)lds;
    const int q = blockIdx.x;
    if (q < 4 * parts) k2_gradient(a, pl, (bf16_t*)(pl + 8 * 34 * kD2W), q % parts, parts, 8 * (q / parts));
    else dy1_strip(a, pl, (float*)(pl + 32 * 18 * kD2W), q - 4 * parts);
}

// ------------------------------------------------------------------ backward of the first layer
// A workgroup takes every gridDim.x-th set: dy1 as one bfloat16 plane per
// channel in LDS.  dx0: each wave sums 8 of the 64 channels, 16 taps a
// matrix instruction, and the eight sums are added in order.  The K1
// gradient (k = the set's 16 input pixels) stays in registers.
__global__ __launch_bounds__(512) void back1_kernel(const TrainArgs a) {
    __shared__ __align__(16) uint32_t pl[64 * (kY1T / 2)];
    __shared__ float dx[8 * 256];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bf16_t* plh = (const bf16_t*)pl;
    bf16x4 w[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) w[o] = frag4(a.w.packed + kT1b, 8 * wave + o, lane);
    f32x4 g[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) g[o] = kZero4;
    for (int b = blockIdx.x; b < a.B; b += gridDim.x) {
        load_transposed<512, 256, 64, kY1T / 2>(a.w.dy1 + (size_t)b * 256 * 64, pl, tid);
        f32x4 xv;   // channel lr of input pixels 4 lq .. 4 lq + 3
#pragma unroll
        for (int v = 0; v < 4; ++v) xv[v] = a.w.x0[((size_t)b * 16 + 4 * lq + v) * 16 + lr];
        const bf16x4 xt = round4(xv);
        __syncthreads();
        f32x4 d = kZero4;
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const bf16_t* p = plh + (8 * wave + o) * kY1T;
            // taps 4 lq .. + 3 of input pixel lr = (i, j): row 4 i + lq, columns 4 j ..
            d = mma16(w[o], lds4(p + (4 * (lr >> 2) + lq) * 16 + 4 * (lr & 3)), d);
            // tap lr of the input pixels (lq, 0..3)
            const bf16_t* q = p + (4 * lq + (lr >> 2)) * 16 + (lr & 3);
            g[o] = mma16(xt, bf16x4{(short)q[0], (short)q[4], (short)q[8], (short)q[12]}, g[o]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) dx[wave * 256 + lr * 16 + 4 * lq + v] = d[v];   // [pixel][channel]
        __syncthreads();
        if (tid < 256) {
            float v = 0.f;
            for (int q = 0; q < 8; ++q) v += dx[q * 256 + tid];
            a.w.dx0[(size_t)b * 256 + tid] = v;
            const size_t f = (size_t)b * 256 + (tid % 16) * 16 + tid / 16;
            a.w.dh2[f] = a.w.h2[f] > 0.f ? v : 0.f;
        }
    }
    float* part = a.w.p1 + (size_t)blockIdx.x * kPart1;
#pragma unroll
    for (int o = 0; o < 8; ++o)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[(4 * lq + v) * 1024 + (8 * wave + o) * 16 + lr] = g[o][v];
}

// dh1 = (dh2 W2^T) masked by h1: 16 sets by 64 columns a workgroup, each
// column tile the sum of its two halves of k.
__global__ __launch_bounds__(256) void back_mlp_kernel(const TrainArgs a) {
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = ((int)blockIdx.x / 4) * 16, n = (((int)blockIdx.x % 4) * 4 + wave) * 16 + lr;
    bf16x4 w[16];
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) w[ks] = frag4(a.w.packed + kT2w, ((int)blockIdx.x % 4 * 4 + wave) * 16 + ks, lane);
    __shared__ __align__(16) bf16_t ds[16 * 264];
    f32x4 dv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // set 4 q + tid / 64, four features a thread
        const int b = min(b0 + 4 * q + wave, a.B - 1);
        dv[q] = load4(a.w.dh2 + (size_t)b * 256 + 4 * lane);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) *(bf16x4*)(ds + (4 * q + wave) * 264 + 4 * lane) = round4(dv[q]);
    __syncthreads();
    const bf16_t* p = ds + lr * 264 + 4 * lq;
    f32x4 d0 = kZero4, d1 = kZero4;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        d0 = mma16(lds4(p + 16 * ks), w[ks], d0);
        d1 = mma16(lds4(p + 16 * ks + 128), w[ks + 8], d1);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int b = b0 + 4 * lq + v;
        if (b < a.B) {
            const size_t f = (size_t)b * 256 + n;
            a.w.dh1[f] = a.w.h1[f] > 0.f ? d0[v] + d1[v] : 0.f;
        }
    }
}

// ------------------------------------------------------------------ gradients out
// The linear layers' weight and bias gradients, and every sum of partial
// sums: segments of `n` values with `parts` partial sums each (`stride`
// floats apart), summed by 256 / cols threads a value in a fixed order.
struct Segment {
    const float* src;
    float* dst;
    int n, parts, stride, cols, block0;
    float div;      // the loss: the sum divided by the number of pixels
};
constexpr int kSegments = 11;
struct FinishArgs {
    Segment seg[kSegments];
    int seg_blocks;             // W2 (4 tiles a block) and W1 come after them
};

__global__ __launch_bounds__(256) void finish_kernel(const TrainArgs a, const FinishArgs f, float* G, const Adam adam) {
    __shared__ float red[256];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = blockIdx.x;
    if (blk >= f.seg_blocks) {
        // x^T d over the sets, one 16 x 16 tile a wave: W2 (h1, dh2), W1 (u, dh1)
        const int t = (blk - f.seg_blocks) * 4 + wave;
        const bool first = t >= 256;
        const int i = first ? lr : (t / 16) * 16 + lr, j = (t % 16) * 16 + lr;
        const float *x = first ? a.w.u : a.w.h1, *d = first ? a.w.dh1 : a.w.dh2;
        const int xw = first ? 4 : 256;
        f32x4 g = kZero4;
        for (int b0 = 0; b0 < a.B; b0 += 64) {   // four products' operands under way at once
            f32x4 xv[4], dv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int b = b0 + 16 * q + 4 * lq + v;
                    xv[q][v] = b < a.B && i < xw ? x[(size_t)b * xw + i] : 0.f;
                    dv[q][v] = b < a.B ? d[(size_t)b * 256 + j] : 0.f;
                }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (b0 + 16 * q < a.B) g = mma16(round4(xv[q]), round4(dv[q]), g);
        }
        float* dst = G + (first ? a.L.W1 : a.L.W2);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = first ? 4 * lq + v : (t / 16) * 16 + 4 * lq + v;
            if (row < xw) {
                dst[row * 256 + j] = g[v];
                if (adam.p) adam.update(dst - G + row * 256 + j, g[v]);
            }
        }
        return;
    }
    int q = 0;
    while (q + 1 < kSegments && blk >= f.seg[q + 1].block0) ++q;
    const Segment s = f.seg[q];
    const int c = tid % s.cols, slice = tid / s.cols, slices = 256 / s.cols;
    const int e = (blk - s.block0) * s.cols + c;
    float sum = 0.f;
    if (e < s.n) {
        const float* p = s.src + e;
        int k = slice;
        for (; k + 7 * slices < s.parts; k += 8 * slices) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p[(size_t)(k + i * slices) * s.stride];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += v[i];
        }
        for (; k < s.parts; k += slices) sum += p[(size_t)k * s.stride];
    }
    red[tid] = sum;
    __syncthreads();
    for (int w = 128; w >= s.cols; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid < s.cols && e < s.n) {
        s.dst[e] = s.div != 0.f ? red[tid] / s.div : red[tid];
        if (adam.p && s.div == 0.f) adam.update(s.dst - G + e, red[tid]);
    }
}

}  // namespace

WS carve(void* base, int B) {
    WS w;
    size_t o = 0;
    auto take = [&](size_t nfloat) {
        float* p = base ? (float*)((char*)base + o) : nullptr;
        o += ((nfloat * sizeof(float) + 255) / 256) * 256;
        return p;
    };
    const size_t b = (size_t)B;
    w.u = take(b * 4);
    w.h1 = take(b * 256);
    w.h2 = take(b * 256);
    w.x0 = take(b * 256);
    w.y1 = take(b * 256 * 64);
    w.y2 = take(b * 1024 * 32);
    w.y3 = take(b * 4096 * 16);
    w.logits = take(b * kImg * kImg);
    w.dlogits = take(b * kImg * kImg);
    w.dy3 = take(b * 4096 * 16);
    w.dy2 = take(b * 1024 * 32);
    w.dy1 = take(b * 256 * 64);
    w.dx0 = take(b * 256);
    w.dh2 = take(b * 256);
    w.dh1 = take(b * 256);
    w.p34 = take(8 * b * kPart34);
    w.p3 = take((size_t)std::min(4 * B, kParts3) * kPart3);
    w.pc1 = take(2 * b * 64);
    w.p2 = take((size_t)std::min(B, kParts2) * kPart2);
    w.p1 = take((size_t)std::min(B, kParts1) * kPart1);
    w.packed = (bf16_t*)take(((size_t)kTrainPacked + 1) / 2);
    w.x0h = (bf16_t*)take(b * 128);
    w.bytes = o;
    return w;
}

hipError_t loss_grad(const float* P, const kl_c64* ta, const kl_c64* tb, const uint8_t* targets, int B, float* G,
                     float* loss, const Adam& adam, const WS& w, hipStream_t s) {
    const TrainArgs a{P, ta, tb, targets, w, layout(), B, sum_chunk(1024 * B, 16), sum_chunk(256 * B, 32)};
    const Layout& L = a.L;
    const int set16 = (B + 15) / 16, n3 = std::min(4 * B, kParts3), n2 = std::min(B, kParts2), n1 = std::min(B, kParts1);
    hipLaunchKernelGGL(prologue_kernel, dim3(4 * set16 + 192), dim3(256), 0, s, a, 4 * set16);
    hipLaunchKernelGGL(conv12_kernel, dim3(4 * B), dim3(256), 0, s, a);
    hipLaunchKernelGGL(conv34_kernel, dim3(8 * B), dim3(512), 0, s, a);
    hipLaunchKernelGGL(back3_kernel, dim3(n3), dim3(512), 0, s, a);
    hipLaunchKernelGGL(back2_kernel, dim3(2 * B + 4 * n2), dim3(512), 0, s, a, n2);
    hipLaunchKernelGGL(back1_kernel, dim3(n1), dim3(512), 0, s, a);
    hipLaunchKernelGGL(back_mlp_kernel, dim3(4 * set16), dim3(256), 0, s, a);
    FinishArgs f{};
    int nseg = 0, blocks = 0;
    auto add = [&](const float* src, float* dst, int n, int parts, int stride, int cols, float div = 0.f) {
        f.seg[nseg++] = {src, dst, n, parts, stride, cols, blocks, div};
        blocks += (n + cols - 1) / cols;
    };
    // many values of few partial sums take many columns a block, few values of many the reverse
    add(w.p2, G + L.K2, kPart2, n2, kPart2, 64);
    add(w.p1, G + L.K1, kPart1, n1, kPart1, 64);
    add(w.p3, G + L.K3, 32 * 256, n3, kPart3, 32);
    add(w.p3 + 32 * 256, G + L.c2, 32, n3, kPart3, 8);
    add(w.p34 + 32, G + L.K4, 256, 8 * B, kPart34, 16);
    add(w.p34 + 2, G + L.c3, 16, 8 * B, kPart34, 2);
    add(w.p34 + 1, G + L.c4, 1, 8 * B, kPart34, 1);
    add(w.p34, loss, 1, 8 * B, kPart34, 1, (float)((int64_t)B * kImg * kImg));
    add(w.pc1, G + L.c1, 64, 2 * B, 64, 8);
    add(w.dh2, G + L.b2, 256, B, 256, 32);
    add(w.dh1, G + L.b1, 256, B, 256, 32);
    f.seg_blocks = blocks;
    hipLaunchKernelGGL(finish_kernel, dim3(blocks + 64 + 4), dim3(256), 0, s, a, f, G, adam);
    return hipGetLastError();
}

}  // namespace sur
}  // namespace kl
