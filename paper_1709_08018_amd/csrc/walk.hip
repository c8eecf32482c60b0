// walk.hip -- the probabilistic approach of Section 4: random walks on the
// group, one orbit per walker, drawn into the density image.
//
// The paper describes this approach only in words: one word grows as
// generators are appended through random picks under some probability law,
// and the orbit of a point under it is drawn.  Here a walker takes a
// uniform first letter c_0, starts at that generator's attracting fixed
// point, and at step k picks c_k uniformly among the three letters that do
// not undo c_{k-1} (so the word stays reduced) and maps its point:
// z_k = G_{c_k}(z_{k-1}).  z_k is then the value of the reduced word
// c_k ... c_1 c_0 from the fixed point of its last letter (Section 1).
// After burn_in steps the walker draws its next n_steps points.  The
// commutator "boost" of the Fig. 3 caption is not applied.
//
// Random numbers: Philox4x64-10 (Salmon, Moraes, Dror, Shaw, "Parallel
// random numbers: as easy as 1, 2, 3", SC'11), counter-based, so that any
// walker's stream is reached without running the others.  Walker w's k-th
// 32-bit value is half k % 2 (low first) of output (k % 8) / 2 of the block
// at the counter (k / 8, w, 0, 0) under the key (seed, 0).  c_0 is the top
// two bits of value 0; c_k (k >= 1) is the floor(3 x / 2^32)-th letter, in
// code order, other than the inverse of c_{k-1}.
//
// Kernel: one thread per walker.  A Philox block gives the thread its next
// eight decisions; the point moves as a homogeneous pair (u : v), the four
// maps read from LDS, rescaled by a power of two (exact) every eight steps;
// each drawn point is u / v, folded into pixel coordinates and binned with
// the renderer's rule (0 <= px < W, 0 <= py < H as IEEE comparisons, NaN and
// infinity outside).  The points of a walk jump across the limit set, so
// there are no runs to merge, and a global atomic per point (walk_kernel)
// costs a cache line per lane.  The binned path (walk_bin_kernel,
// walk_tile_hist_kernel) instead sorts each workgroup's points of one Philox
// block (8 steps) by image tile of 2^15 bins in LDS and writes them out as
// 16-bit offsets within their tiles; a second kernel counts each tile's
// offsets in an LDS histogram and adds its non-zero bins to the image.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kl_internal.hpp"

namespace kl {

namespace {

constexpr uint64_t kPhiloxM0 = 0xD2E7470EE14C6C93ull, kPhiloxM1 = 0xCA5A826395121157ull;
constexpr uint64_t kPhiloxW0 = 0x9E3779B97F4A7C15ull, kPhiloxW1 = 0xBB67AE8584CAA73Bull;

// The 128-bit product a m of 64-bit words, from the four 32 x 32-bit
// partial products (each a multiply-add into 64 bits that cannot overflow):
// both halves come from the same four multiply-adds.
template <uint64_t M>
__device__ __forceinline__ void mul128(uint64_t a, uint64_t& hi, uint64_t& lo) {
    constexpr uint32_t m0 = (uint32_t)M, m1 = (uint32_t)(M >> 32);
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
    const uint64_t p0 = (uint64_t)a0 * m0;
    const uint64_t p1 = (uint64_t)a0 * m1 + (p0 >> 32);
    const uint64_t p2 = (uint64_t)a1 * m0 + (uint32_t)p1;
    hi = (uint64_t)a1 * m1 + (p1 >> 32) + (p2 >> 32);
    lo = (p2 << 32) | (uint32_t)p0;
}

// Ten Philox4x64 rounds: each takes the 128-bit products of words 0 and 2
// with the two multipliers and mixes their halves with words 1 and 3 and
// the key; the key advances by the two Weyl constants between rounds.
__device__ __forceinline__ void philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                              uint64_t k1, uint64_t out[4]) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            k0 += kPhiloxW0;
            k1 += kPhiloxW1;
        }
        uint64_t hi0, lo0, hi1, lo1;
        mul128<kPhiloxM0>(c0, hi0, lo0);
        mul128<kPhiloxM1>(c2, hi1, lo1);
        const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// bin of pixel coordinates, the renderer's rule; kWalkOutside when outside
constexpr uint32_t kWalkOutside = 0xFFFFFFFFu;

// FP32: on the floors, saturating int32 (v_cvt_flr_i32_f32; NaN to 0, so NaNs
// are told apart by an ordered comparison), as the renderer bins
__device__ __forceinline__ int walk_floor(float x) {
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ uint32_t walk_bin(float px, float py, uint32_t W, uint32_t H) {
    const uint32_t col = (uint32_t)walk_floor(px), row = (uint32_t)walk_floor(py);
    const bool ok = (col < W) & (row < H) & !__builtin_isunordered(px, py);
    return ok ? __umul24(row, W) + col : kWalkOutside;
}

__device__ __forceinline__ uint32_t walk_bin(double px, double py, uint32_t W, uint32_t H) {
    const bool ok = (px >= 0.0) & (px < (double)W) & (py >= 0.0) & (py < (double)H);
    return ok ? (uint32_t)__builtin_floor(py) * W + (uint32_t)__builtin_floor(px) : kWalkOutside;
}

__device__ __forceinline__ float wabs(float x) { return __builtin_fabsf(x); }
__device__ __forceinline__ double wabs(double x) { return __builtin_fabs(x); }
__device__ __forceinline__ float wmax(float x, float y) { return __builtin_fmaxf(x, y); }
__device__ __forceinline__ double wmax(double x, double y) { return __builtin_fmax(x, y); }
__device__ __forceinline__ float wldexp(float x, int e) { return __builtin_ldexpf(x, e); }
__device__ __forceinline__ double wldexp(double x, int e) { return __builtin_ldexp(x, e); }
__device__ __forceinline__ int wexp(float x) { return __builtin_amdgcn_frexp_expf(x); }
__device__ __forceinline__ int wexp(double x) { return __builtin_amdgcn_frexp_exp(x); }

// (u : v) scaled by the power of two that brings its largest component into
// [0.5, 1); exact, and the point u / v is unchanged
template <typename T>
__device__ __forceinline__ void walk_rescale(cpx<T>& u, cpx<T>& v) {
    const T m = wmax(wmax(wabs(u.re), wabs(u.im)), wmax(wabs(v.re), wabs(v.im)));
    if (m > T(0) && m < T(INFINITY)) {
        const int e = -wexp(m);
        u = {wldexp(u.re, e), wldexp(u.im, e)};
        v = {wldexp(v.re, e), wldexp(v.im, e)};
    }
}

// 1 / x as the renderer takes it: v_rcp_f32 in FP32 (within an ulp), and in
// FP64 v_rcp_f64 refined by two Newton steps r <- r + r (1 - x r), a
// full-precision reciprocal.  x = 0 (a point at infinity) gives infinity or
// NaN, and the point is dropped.
__device__ __forceinline__ float walk_recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double walk_recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma_(-x, r, 1.0);
    r = fma_(r, e, r);
    e = fma_(-x, r, 1.0);
    return fma_(r, e, r);
}

// The four maps and the seeds (u : v) in LDS, one entry per letter.
template <typename T>
struct WalkMaps {
    mat<T> G[4];
    cpx<T> SU[4], SV[4];
};

template <typename T>
__device__ __forceinline__ void load_walk_maps(const WalkJob& j, WalkMaps<T>& m) {
    if (threadIdx.x < 4) {
        const m64& g = j.gens.g[threadIdx.x];
        m.G[threadIdx.x] = {{(T)g.a.re, (T)g.a.im}, {(T)g.b.re, (T)g.b.im}, {(T)g.c.re, (T)g.c.im},
                            {(T)g.d.re, (T)g.d.im}};
        const bool inf = (j.gens.inf_mask >> threadIdx.x) & 1u;
        m.SU[threadIdx.x] = inf ? cpx<T>{T(1), T(0)} : cpx<T>{(T)j.gens.fix[threadIdx.x].re, (T)j.gens.fix[threadIdx.x].im};
        m.SV[threadIdx.x] = inf ? cpx<T>{T(0), T(0)} : cpx<T>{T(1), T(0)};
    }
}

// One walker's state, and its step k (x: value k of its stream), k > burn_in
// giving the drawn point in the window's pixel coordinates.
template <typename T>
struct Walker {
    cpx<T> u, v;
    int prev;
};

template <typename T>
struct WalkFold {
    T s, ox, oy, an;
};

template <typename T>
__device__ __forceinline__ int walk_letter(const Walker<T>& w, uint32_t k, uint32_t x) {
    if (k == 0) return (int)(x >> 30);
    const int t = (int)__umulhi(x, 3u);
    return t + (t >= (w.prev ^ 2));
}

template <typename T>
__device__ __forceinline__ void walk_step(Walker<T>& w, const WalkMaps<T>& m, uint32_t k, int c) {
    if (k == 0) {
        w.u = m.SU[c];
        w.v = m.SV[c];
    } else {
        const mat<T> g = m.G[c];
        const cpx<T> nu = cfma(g.a, w.u, cmul(g.b, w.v));
        const cpx<T> nv = cfma(g.c, w.u, cmul(g.d, w.v));
        w.u = nu;
        w.v = nv;
    }
    w.prev = c;
}

// z = u / v, then the window's affine map s z + o (x anisotropy on the real part)
template <typename T>
__device__ __forceinline__ void walk_pixel(const Walker<T>& w, const WalkFold<T>& f, T& px, T& py) {
    const T n2 = fma_(w.v.re, w.v.re, w.v.im * w.v.im);
    const T rc = walk_recip(n2);
    const T zr = fma_(w.u.re, w.v.re, w.u.im * w.v.im) * rc;
    const T zi = fma_(w.u.im, w.v.re, -(w.u.re * w.v.im)) * rc;
    px = fma_(f.s, zr, f.ox) * f.an;
    py = fma_(f.s, zi, f.oy);
}

template <typename T>
__device__ __forceinline__ WalkFold<T> walk_fold(const WalkJob& j) {
    return {(T)j.fold.s, (T)j.fold.o.re, (T)j.fold.o.im, (T)j.fold.aniso};
}

// Letters, points or a render with one global atomic per point.  A small walk
// is bound by its serial chain (letter, matrix from LDS, product), so a block
// of eight steps that are all drawn goes without conditions between them,
// which lets the letters and matrices of later steps be fetched during
// earlier products.  1,754 walkers of 118 steps: 36.2 us in FP64 and 31.1
// in FP32, with a condition per step 45.1 and 41.5.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void walk_kernel(const WalkJob j) {
    __shared__ WalkMaps<T> m;
    load_walk_maps(j, m);
    __syncthreads();
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t drop = 0;   // at most n_steps
    if (tid < j.n_walkers) {
        const uint32_t n_total = 1 + j.burn_in + j.n_steps;
        const WalkFold<T> f = walk_fold<T>(j);
        Walker<T> w = {{T(0), T(0)}, {T(1), T(0)}, 0};
        for (uint64_t blk = 0; blk * 8 < n_total; ++blk) {   // 64 bits: n_total may be 2^32 - 1
            const uint32_t k0 = (uint32_t)(blk * 8);
            uint64_t r[4];
            philox4x64_10(blk, j.first_walker + tid, 0, 0, j.seed, 0, r);
            // inner: every step of the block is drawn (and none is the first)
            auto steps = [&](auto inner) {
#pragma unroll
                for (uint32_t i = 0; i < 8; ++i) {
                    const uint32_t k = inner.value ? 1u : k0 + i;
                    if (!inner.value && i >= n_total - k0) continue;
                    const int c = walk_letter(w, k, (uint32_t)(r[i >> 1] >> (32 * (i & 1))));
                    if (MODE == kWalkLetters) {
                        w.prev = c;
                        j.letters[tid * n_total + k0 + i] = (uint8_t)c;
                        continue;
                    }
                    walk_step(w, m, k, c);
                    if (!inner.value && k <= j.burn_in) continue;
                    T px, py;
                    walk_pixel(w, f, px, py);
                    if (MODE == kWalkEval) {
                        j.z_out[tid * j.n_steps + (k0 + i - j.burn_in - 1)] = {(double)px, (double)py};
                    } else {
                        const uint32_t b = walk_bin(px, py, j.W, j.H);
                        if (b != kWalkOutside) atomicAdd(j.image + b, 1u);
                        else ++drop;
                    }
                }
            };
            if (k0 > j.burn_in && n_total - k0 >= 8) steps(std::true_type{});
            else steps(std::false_type{});
            if (MODE != kWalkLetters) walk_rescale(w.u, w.v);
        }
    }
    if (MODE == kWalkRender && j.dropped) {
        uint64_t sum = drop;
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if ((threadIdx.x & 63) == 0 && sum) atomicAdd((unsigned long long*)j.dropped, (unsigned long long)sum);
    }
}

// ---- binned render
// One region per (workgroup, Philox block): its points in the window as
// offsets within their tiles, tile by tile (ids, kRegion slots a region),
// and where each tile's offsets start (starts, T + 1 entries a region:
// starts[T] is the region's count).
//
// A point takes one LDS atomic, whose old value is its rank among its tile's
// points; after a scan of the tiles' counts, first point plus rank is its
// place.  Three barriers a region: the counters alternate, so one set is
// cleared while the other is read.  What bounds it: VALU issue (some 90
// instructions a point, 28 of them the Philox rounds, whose 64-bit products
// issue at a quarter of the rate; sums with carries in place of their chained
// addends took 7% longer).  2^26 points in FP32: 137 us (traced in a long run
// of calls, with the histogram's 50 the call's 187); with the bins staged in
// LDS eight words apart (8-way bank conflicts), a second atomic and five
// barriers 189.  Workgroups of 256 walkers, which walks of some 2^18 steps take
// (walk_binned_layout), need 7% less here, but their regions are half as long
// and the histogram kernel pays for it (64 us against 50).
template <typename T>
constexpr int kWalkWaves = std::is_same<T, float>::value ? 6 : 5;   // per SIMD, without spills

template <typename T, uint32_t WALKERS>
__global__ __launch_bounds__(WALKERS) __attribute__((amdgpu_waves_per_eu(kWalkWaves<T>))) void walk_bin_kernel(
    const WalkJob j, uint16_t* __restrict__ ids, uint32_t* __restrict__ starts, uint32_t T_tiles, uint32_t n_chunks) {
    constexpr uint32_t kRegion = WALKERS * kWalkChunk;   // slots of a region
    __shared__ WalkMaps<T> m;
    __shared__ __align__(4) uint16_t sorted[kRegion];
    __shared__ uint32_t cnt[2][kMaxWalkTiles], base[kMaxWalkTiles + 1];
    load_walk_maps(j, m);
    for (uint32_t t = threadIdx.x; t < kMaxWalkTiles; t += blockDim.x) cnt[0][t] = 0;
    __syncthreads();
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    {   // the image is cleared while the walkers start; only the histograms add to it
        const uint64_t n = (uint64_t)gridDim.x * blockDim.x;
        const uint64_t n4 = ((uintptr_t)j.image & 15) == 0 ? j.clear_bins / 4 : 0;
        for (uint64_t i = tid; i < n4; i += n) ((uint4*)j.image)[i] = make_uint4(0, 0, 0, 0);
        for (uint64_t i = 4 * n4 + tid; i < j.clear_bins; i += n) j.image[i] = 0;
    }
    const bool active = tid < j.n_walkers;   // the others step along on the first walker's stream
    const uint64_t walker = j.first_walker + (active ? tid : 0);
    const uint32_t n_total = 1 + j.burn_in + j.n_steps;
    const WalkFold<T> f = walk_fold<T>(j);
    Walker<T> w = {{T(0), T(0)}, {T(1), T(0)}, 0};
    const uint32_t W = active ? j.W : 0u;    // ... and every point of theirs is outside
    uint32_t drop = 0;   // at most n_steps
    uint64_t region = (uint64_t)blockIdx.x * n_chunks;
    uint32_t par = 0;
    for (uint64_t blk = 0; blk * kWalkChunk < n_total; ++blk) {   // 64 bits: n_total may be 2^32 - 1
        const uint32_t k0 = (uint32_t)(blk * kWalkChunk);
        uint64_t r[4];
        philox4x64_10(blk, walker, 0, 0, j.seed, 0, r);
        uint32_t bin[kWalkChunk], rank[kWalkChunk];
        // inner: every step of the block is drawn (and none is the first)
        auto steps = [&](auto inner) {
#pragma unroll
            for (uint32_t i = 0; i < kWalkChunk; ++i) {
                const uint32_t k = inner.value ? 1u : k0 + i;   // uniform: every walker takes the same steps
                bin[i] = kWalkOutside;
                rank[i] = 0;
                if (!inner.value && i >= n_total - k0) continue;
                walk_step(w, m, k, walk_letter(w, k, (uint32_t)(r[i >> 1] >> (32 * (i & 1)))));
                if (!inner.value && k <= j.burn_in) continue;
                T px, py;
                walk_pixel(w, f, px, py);
                bin[i] = walk_bin(px, py, W, j.H);
                if (bin[i] != kWalkOutside) rank[i] = atomicAdd(&cnt[par][bin[i] >> kWalkTileBits], 1u);
                else ++drop;
            }
        };
        if (k0 > j.burn_in && n_total - k0 >= kWalkChunk) steps(std::true_type{});
        else steps(std::false_type{});
        walk_rescale(w.u, w.v);
        if ((blk + 1) * kWalkChunk <= (uint64_t)j.burn_in + 1) continue;   // no drawn step yet
        __syncthreads();
        if (threadIdx.x < 64) {
            // exclusive scan of the counts by one wave, base[T] the total
            uint32_t carry = 0;
            for (uint32_t t0 = 0; t0 < T_tiles; t0 += 64) {
                const uint32_t t = t0 + threadIdx.x;
                const uint32_t c = t < T_tiles ? cnt[par][t] : 0u;
                uint32_t x = c;
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t y = __shfl_up(x, off, 64);
                    if ((int)threadIdx.x >= off) x += y;
                }
                if (t < T_tiles) base[t] = carry + x - c;
                carry += __shfl(x, 63, 64);
            }
            if (threadIdx.x == 0) base[T_tiles] = carry;
        } else {
            for (uint32_t t = threadIdx.x - 64; t < T_tiles; t += blockDim.x - 64) cnt[par ^ 1][t] = 0;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kWalkChunk; ++i)
            if (bin[i] != kWalkOutside)
                sorted[base[bin[i] >> kWalkTileBits] + rank[i]] = (uint16_t)(bin[i] & (kWalkTileBins - 1));
        __syncthreads();
        const uint32_t n2 = (base[T_tiles] + 1) / 2;   // whole dwords: a region's slots are its own
        uint32_t* out = (uint32_t*)(ids + region * kRegion);
        for (uint32_t i = threadIdx.x; i < n2; i += blockDim.x) out[i] = ((const uint32_t*)sorted)[i];
        uint32_t* st = starts + region * (T_tiles + 1);
        for (uint32_t t = threadIdx.x; t <= T_tiles; t += blockDim.x) st[t] = base[t];
        ++region;
        par ^= 1;
    }
    if (j.dropped) {
        uint64_t sum = active ? drop : 0u;
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if ((threadIdx.x & 63) == 0 && sum) atomicAdd((unsigned long long*)j.dropped, (unsigned long long)sum);
    }
}

// The tile histogram reads a region's offsets of one tile (its segment) in
// 16-byte chunks of 8 offsets, 8 lanes to a region, so that one load
// instruction of a wave covers the first 64 offsets of 8 regions; a wave
// loads the first chunks of kHistPasses such groups of 8 regions before
// counting them, and loads the segment bounds of its next 64 regions while
// it counts the current ones.
constexpr uint32_t kHistLanes = 8;    // lanes per region
constexpr uint32_t kHistPasses = 4;   // groups of 8 regions loaded before counting

// count the offsets of chunk c (offsets 8c .. 8c + 7 of the region) that
// lie in the segment [a, b)
__device__ __forceinline__ void hist_chunk(uint32_t* hist, uint4 v, uint32_t c, uint32_t a, uint32_t b) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (uint32_t e = 0; e < 8; ++e) {
        const uint32_t i = 8 * c + e;
        if (i >= a && i < b) atomicAdd(&hist[(w[e / 2] >> (16 * (e % 2))) & 0xFFFFu], 1u);
    }
}

// Which tile a workgroup counts, and which of the tile's `of` equal shares of
// the regions.  Walks crowd into some tiles (the fullest of Fig. 3's window
// holds 3.4 times the mean, four of 32 are empty), so the workgroups are dealt
// to the tiles by the rounds that up to kHistSamples regions, spread over all,
// take: every tile gets one workgroup, the other gridDim.x - T in proportion
// (rounded down; workgroups left over return at once).
constexpr uint32_t kHistSamples = 64;
struct HistShare {
    uint32_t tile, part, of;   // of = 0: no share
};

__device__ __forceinline__ HistShare hist_share(const uint32_t* __restrict__ starts, uint64_t n_regions, uint32_t T) {
    __shared__ uint32_t weight[kMaxWalkTiles];
    __shared__ HistShare share;
    for (uint32_t t = threadIdx.x; t < T; t += blockDim.x) weight[t] = 0;
    __syncthreads();
    const uint32_t samples = n_regions < kHistSamples ? (uint32_t)n_regions : kHistSamples;
    for (uint32_t i = threadIdx.x; i < samples * T; i += blockDim.x) {
        const uint32_t q = i / T, t = i - q * T;
        const uint32_t* st = starts + (n_regions * q / samples) * (T + 1) + t;
        // a region costs one round of its lanes' chunks (64 offsets) at least
        const uint32_t c = st[1] - st[0], rounds = (c + 63) / 64;
        atomicAdd(&weight[t], rounds ? rounds : 1u);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t lane = threadIdx.x;
        uint32_t sum = 0;
        for (uint32_t t = lane; t < T; t += 64) sum += weight[t];
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) share = {0, 0, 0};
        uint32_t carry = 0;
        for (uint32_t t0 = 0; t0 < T; t0 += 64) {
            const uint32_t t = t0 + lane;
            const uint32_t n = t < T ? 1u + (uint32_t)((uint64_t)weight[t] * (gridDim.x - T) / (sum ? sum : 1u)) : 0u;
            uint32_t x = n;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t y = __shfl_up(x, off, 64);
                if ((int)lane >= off) x += y;
            }
            const uint32_t lo = carry + x - n;
            if (blockIdx.x >= lo && blockIdx.x - lo < n) share = {t, blockIdx.x - lo, n};
            carry += __shfl(x, 63, 64);
        }
    }
    __syncthreads();
    return share;
}

// One tile over a share of the regions: every offset counted in an LDS
// histogram, then each non-zero bin added to the image.  What bounds it: the
// latency of the offsets' loads and the LDS atomics, sixteen waves a CU (the
// histogram takes 128 KB).  2^26 points: 50 us; with an equal number of
// workgroups for every tile, and regions of 256 walkers, 63.
template <uint32_t WALKERS>
__global__ __launch_bounds__(1024) void walk_tile_hist_kernel(const uint16_t* __restrict__ ids,
                                                              const uint32_t* __restrict__ starts,
                                                              uint64_t n_regions, uint32_t T_tiles,
                                                              uint32_t* __restrict__ image) {
    constexpr uint32_t kRegion = WALKERS * kWalkChunk;
    __shared__ __align__(16) uint32_t hist[kWalkTileBins];
    const HistShare share = hist_share(starts, n_regions, T_tiles);
    if (share.of == 0) return;
    const uint32_t tile = share.tile;
    for (uint32_t i = threadIdx.x; i < kWalkTileBins / 4; i += blockDim.x) ((uint4*)hist)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const uint64_t r0 = n_regions * share.part / share.of, r1 = n_regions * (share.part + 1) / share.of;
    const uint32_t wave = threadIdx.x / 64, lane = threadIdx.x % 64, waves = blockDim.x / 64;
    const uint32_t grp = lane / kHistLanes, sub = lane % kHistLanes;
    // a wave takes a contiguous slice of the regions, 64 at a time; lane l
    // holds the segment bounds [a, b) of region base + l (0, 0 past the slice)
    const uint64_t per = (r1 - r0 + waves - 1) / waves;
    const uint64_t w0 = r0 + wave * per, w1 = w0 + per < r1 ? w0 + per : r1;
    uint32_t na = 0, nb_ = 0;
    if (w0 + lane < w1) {
        const uint32_t* st = starts + (w0 + lane) * (T_tiles + 1);
        na = st[tile];
        nb_ = st[tile + 1];
    }
    for (uint64_t base = w0; base < w1; base += 64) {
        const uint32_t a = na, b = nb_;
        na = 0;
        nb_ = 0;
        if (base + 64 + lane < w1) {
            const uint32_t* st = starts + (base + 64 + lane) * (T_tiles + 1);
            na = st[tile];
            nb_ = st[tile + 1];
        }
        const uint32_t n = w1 - base < 64 ? (uint32_t)(w1 - base) : 64u;
        for (uint32_t j = 0; j < n; j += kHistLanes * kHistPasses) {
            uint4 v[kHistPasses];
            uint32_t aq[kHistPasses], bq[kHistPasses], cq[kHistPasses];
            const uint16_t* seg[kHistPasses];
#pragma unroll
            for (uint32_t q = 0; q < kHistPasses; ++q) {
                const uint32_t r = j + kHistLanes * q + grp;   // < 64
                aq[q] = __shfl(a, (int)r, 64);
                bq[q] = __shfl(b, (int)r, 64);
                cq[q] = aq[q] / 8 + sub;
                seg[q] = ids + (base + r) * kRegion;
                v[q] = 8 * cq[q] < bq[q] ? *(const uint4*)(seg[q] + 8 * cq[q]) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (uint32_t q = 0; q < kHistPasses; ++q)
                if (8 * cq[q] < bq[q]) hist_chunk(hist, v[q], cq[q], aq[q], bq[q]);
            // segments longer than the group's first 8 chunks
#pragma unroll
            for (uint32_t q = 0; q < kHistPasses; ++q)
                for (uint32_t c = cq[q] + kHistLanes; 8 * c < bq[q]; c += kHistLanes)
                    hist_chunk(hist, *(const uint4*)(seg[q] + 8 * c), c, aq[q], bq[q]);
        }
    }
    __syncthreads();
    uint32_t* img = image + (uint64_t)tile * kWalkTileBins;
    for (uint32_t i = threadIdx.x; i < kWalkTileBins; i += blockDim.x) {
        const uint32_t v = hist[i];
        if (v) atomicAdd(img + i, v);
    }
}

}  // namespace

// Walkers go in launches of at most 2^30 (2^22 blocks), each with its
// outputs advanced to its first walker.
hipError_t launch_walk(const WalkJob& j, hipStream_t s) {
    const uint64_t per = 1ull << 30;
    const uint64_t n_total = 1ull + j.burn_in + j.n_steps;
    for (uint64_t off = 0; off < j.n_walkers; off += per) {
        WalkJob c = j;
        c.first_walker = j.first_walker + off;
        c.n_walkers = j.n_walkers - off < per ? j.n_walkers - off : per;
        if (c.letters) c.letters += off * n_total;
        if (c.z_out) c.z_out += off * j.n_steps;
        const unsigned blocks = (unsigned)((c.n_walkers + 255) / 256);
        const bool fp64 = j.precision == KL_PREC_FP64;
        void (*kern)(WalkJob) = j.mode == kWalkLetters ? walk_kernel<float, kWalkLetters>
                                : j.mode == kWalkEval  ? (fp64 ? walk_kernel<double, kWalkEval> : walk_kernel<float, kWalkEval>)
                                                       : (fp64 ? walk_kernel<double, kWalkRender> : walk_kernel<float, kWalkRender>);
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, s, c);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The binned render: walkers in launches of L.blocks workgroups, each launch
// binning its walkers' points (walk_bin_kernel) and then counting them tile by
// tile (walk_tile_hist_kernel), in `buf` (L.bytes bytes).
hipError_t launch_walk_binned(const WalkJob& j, const WalkBinned& L, void* buf, hipStream_t s) {
    if (L.blocks == 0) return hipSuccess;
    const uint32_t T_tiles = walk_tiles(j.W, j.H);
    const uint64_t total_blocks = (j.n_walkers + L.walkers - 1) / L.walkers;
    uint16_t* ids = (uint16_t*)buf;
    uint32_t* starts = (uint32_t*)((unsigned char*)buf + L.off_starts);
    const bool fp64 = j.precision == KL_PREC_FP64;
    void (*bin)(WalkJob, uint16_t*, uint32_t*, uint32_t, uint32_t) =
        L.walkers == kWalkBlock ? (fp64 ? walk_bin_kernel<double, kWalkBlock> : walk_bin_kernel<float, kWalkBlock>)
                                : (fp64 ? walk_bin_kernel<double, kWalkBlockSmall> : walk_bin_kernel<float, kWalkBlockSmall>);
    void (*hist)(const uint16_t*, const uint32_t*, uint64_t, uint32_t, uint32_t*) =
        L.walkers == kWalkBlock ? walk_tile_hist_kernel<kWalkBlock> : walk_tile_hist_kernel<kWalkBlockSmall>;
    // two workgroups for each CU, or for each tile if that is more
    const unsigned hist_blocks = std::max(2u * (unsigned)device_cu_count(), 2u * T_tiles);
    for (uint64_t b0 = 0; b0 < total_blocks; b0 += L.blocks) {
        const uint64_t nb = std::min(total_blocks - b0, L.blocks);
        WalkJob c = j;
        c.first_walker = j.first_walker + b0 * L.walkers;
        c.n_walkers = std::min(j.n_walkers - b0 * L.walkers, nb * L.walkers);
        if (b0) c.clear_bins = 0;
        hipLaunchKernelGGL(bin, dim3((unsigned)nb), dim3(L.walkers), 0, s, c, ids, starts, T_tiles, L.chunks);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(hist, dim3(hist_blocks), dim3(1024), 0, s, ids, starts, nb * L.chunks, T_tiles, j.image);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kl
