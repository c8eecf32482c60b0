// cayley.hip -- gfx950 kernels of libkl for words of an indexed Cayley
// table (Section 5 of the paper): decode, FP64 values and images.
#include <algorithm>

#include "kl_internal.hpp"

namespace kl {

constexpr uint32_t kCayleyOutside = 0xFFFFFFFFu;

// Bin of FP64 pixel coordinates, or kCayleyOutside when outside
// [0, W) x [0, H) or NaN (every comparison with NaN is false).
__device__ __forceinline__ uint32_t cayley_bin(double px, double py, uint32_t W, uint32_t H) {
    const bool ok = (px >= 0.0) & (px < (double)W) & (py >= 0.0) & (py < (double)H);
    const uint32_t col = ok ? (uint32_t)px : 0u;
    const uint32_t row = ok ? (uint32_t)py : 0u;
    return ok ? __umul24(row, W) + col : kCayleyOutside;
}

}  // namespace kl

namespace kl {

// Words of an indexed Cayley table (Section 5): symbols 1..m, states 0..S-1,
// a word x_1..x_d read right to left from state 0 and regular when no step
// lands in state 0 again; words numbered in lexicographic order, x_1 most
// significant.  C[L][s] counts the regular words of length L whose walk
// ends in state s.  A prefix is read after the rest of its word, from the
// state the rest ended in; `good` holds the states from which the prefix so
// far reads without a crash, and the words that begin with it number
// sum over s in good of C[remaining][s].  Choosing the next symbol x
// restricts good to the states s with T(s, x) != 0 and T(s, x) in good.
//
// The word's maps are multiplied left to right in FP64 while it is
// unranked, then applied to the seed: the attracting fixed point of its
// last symbol, or of one symbol for every word.
// 1 / x: v_rcp_f64 refined by two Newton steps r <- r + r (1 - x r), a
// full-precision reciprocal (x = 0 or an infinite x give NaN, a word that
// is dropped)
__device__ __forceinline__ double cayley_recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma_(-x, r, 1.0);
    r = fma_(r, e, r);
    e = fma_(-x, r, 1.0);
    return fma_(r, e, r);
}

// pixel coordinates (or z itself under the identity fold) of the point (num : den)
__device__ inline void cayley_pixel(const CayleyJob& a, c64 num, c64 den, double& px, double& py) {
    const double rc = cayley_recip(fma_(den.re, den.re, den.im * den.im));
    const double re = fma_(num.re, den.re, num.im * den.im) * rc;
    const double im = fma_(num.im, den.re, -(num.re * den.im)) * rc;
    px = fma_(a.fold.s, re, a.fold.o.re) * a.fold.aniso;
    py = fma_(a.fold.s, im, a.fold.o.im);
}

// A tail point (u : v) as stored in a tail table: (y : 1) with y = u / v
// where v != 0 and y is in range, else (u : v) unchanged (a point at or near
// infinity).  Tails stored as (y : 1) take the pole form.
__device__ inline void cayley_tail_normalize(c64& u, c64& v) {
    const double n2 = fma_(v.re, v.re, v.im * v.im);
    const c64 y = {fma_(u.re, v.re, u.im * v.im) / n2, fma_(u.im, v.re, -(u.re * v.im)) / n2};
    if (n2 > 0.0 && y.re <= 0x1p32 && y.re >= -0x1p32 && y.im <= 0x1p32 && y.im >= -0x1p32) {
        u = y;
        v = {1.0, 0.0};
    }
}

// A head's map [[a, b], [c, d]] in pole form, for c != 0:
//   h(y) = P + Q / (y + S),  P = a / c,  S = d / c,  Q = -(a d - b c) / c^2,
// with the pixel fold applied (P <- s P + o, Q <- s Q) and the x anisotropy
// folded into the real part's coefficients, so that with u = y + S
//   px = Px + (ax u.re + bx u.im) / |u|^2,  py = Py + (ay u.re + by u.im) / |u|^2;
// the map itself is kept for the ratio form.
struct CayleyHead {
    m64 M;
    c64 S;
    double Px, Py, ax, bx, ay, by;
    bool pole;
};

__device__ inline CayleyHead cayley_head(const CayleyJob& a, const m64& M) {
    CayleyHead h;
    h.M = M;
    const double cn = fma_(M.c.re, M.c.re, M.c.im * M.c.im);
    const double rn = cayley_recip(cn);
    const c64 ic = {M.c.re * rn, -(M.c.im * rn)};
    const c64 P = cmul(M.a, ic);
    h.S = cmul(M.d, ic);
    const c64 det = {fma_(M.a.re, M.d.re, -(M.a.im * M.d.im)) - fma_(M.b.re, M.c.re, -(M.b.im * M.c.im)),
                     fma_(M.a.re, M.d.im, M.a.im * M.d.re) - fma_(M.b.re, M.c.im, M.b.im * M.c.re)};
    const c64 q = cmul(det, cmul(ic, ic));
    const double s = a.fold.s, an = a.fold.aniso;
    h.Px = fma_(s, P.re, a.fold.o.re) * an;
    h.Py = fma_(s, P.im, a.fold.o.im);
    h.ax = -(s * q.re) * an;
    h.bx = -(s * q.im) * an;
    h.ay = -(s * q.im);
    h.by = s * q.re;
    auto in = [](double x, double lim) { return x <= lim && x >= -lim; };   // false for NaN
    h.pole = cn > 0.0 && cn <= 0x1p1000 && in(h.S.re, 0x1p40) && in(h.S.im, 0x1p40) && in(h.ax, 0x1p80) &&
             in(h.bx, 0x1p80) && in(h.ay, 0x1p80) && in(h.by, 0x1p80) && in(h.Px, 0x1p100) && in(h.Py, 0x1p100);
    return h;
}

// Pole form at the point y.
__device__ __forceinline__ void cayley_pole_word(const CayleyHead& h, c64 y, double& px, double& py) {
    const double ur = y.re + h.S.re, ui = y.im + h.S.im;
    const double rc = cayley_recip(fma_(ur, ur, ui * ui));
    px = fma_(fma_(h.ax, ur, h.bx * ui), rc, h.Px);
    py = fma_(fma_(h.ay, ur, h.by * ui), rc, h.Py);
}

// Run key of a word: the saturating int32 floors of its pixel coordinates,
// (row, column), in the window exactly when both are (cayley_bin's rule).
// v_cvt_i32_f64 maps NaN to 0, so px goes through a maximum with -1, which
// keeps the number: a NaN px is outside.  In the pole form, whose guards keep
// every other factor finite, px and py are NaN together (with the
// reciprocal); elsewhere the caller checks.
constexpr uint64_t kCayleyOutsideKey = ~0ull;
__device__ __forceinline__ int cayley_floor(double x) {
    int r;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(__builtin_floor(x)));
    return r;
}
__device__ __forceinline__ uint64_t cayley_pole_key(double px, double py) {
    return (uint64_t)(uint32_t)cayley_floor(__builtin_fmax(px, -1.0)) | ((uint64_t)(uint32_t)cayley_floor(py) << 32);
}

// Pixel coordinates of head . tail from the tail's stored point (u : v): the
// pole form where the head has one and the point is (y : 1), else the ratio
// form.  Render and eval both come here, so their values agree bit for bit.
__device__ inline void cayley_word(const CayleyJob& a, const CayleyHead& h, c64 u, c64 v, double& px, double& py) {
    if (h.pole && v.re == 1.0 && v.im == 0.0) {
        cayley_pole_word(h, u, px, py);
    } else {
        cayley_pixel(a, cfma(h.M.a, u, cmul(h.M.b, v)), cfma(h.M.c, u, cmul(h.M.d, v)), px, py);
    }
}

// symbol j (0-based, x - 1) of a word packed 3 bits each into lo (0..20) and hi (21..39)
__device__ __forceinline__ int packed_symbol(uint64_t lo, uint64_t hi, int j) {
    return (int)((j < 21 ? lo >> (3 * j) : hi >> (3 * (j - 21))) & 7u);
}

// Wave-level barrier for LDS written and read by the lanes of one wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Counts of the regular words by length and end state, C[L * stride + s]
// for L = 0..D, from the table copied to LDS (TB): A[t * S + s] counts the
// symbols that take state s to state t != 0, and C[L][t] = sum over s of
// A[t][s] C[L - 1][s].  The first wave forms the lengths one after another
// (one lane per state); the block is synchronised on return.
__device__ inline void cayley_counts(const uint8_t* TB, uint8_t* A, uint64_t* C, int stride, int S, int m, int D) {
    for (int i = threadIdx.x; i < S * S; i += blockDim.x) {
        const int t = i / S, s = i - t * S;
        int n = 0;
        if (t != 0)
            for (int x = 1; x <= m; ++x) n += TB[s * (m + 1) + x] == t ? 1 : 0;
        A[i] = (uint8_t)n;
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)kWave) {
        const int t = threadIdx.x;
        if (t < S) C[t] = t == 0 ? 1 : 0;
        wave_sync();
        for (int L = 1; L <= D; ++L) {
            if (t < S) {
                uint64_t n = 0;
                for (int s = 0; s < S; ++s) n += (uint64_t)A[t * S + s] * C[(L - 1) * stride + s];
                C[L * stride + t] = n;
            }
            wave_sync();
        }
    }
    __syncthreads();
}

// The good sets reachable from the set of all states form a deterministic
// automaton (next_set); CM[L][g] = sum over s in set g of C[L][s] counts the
// words that begin with a prefix of good set g and have L symbols to go.
// Choosing a symbol is then two table reads per candidate.  A word's
// symbols are packed 3 bits each (x - 1) into two registers.
//
// Decode, eval, and renders of words shorter than r (launch_cayley sends a
// render's words of depth >= r to cayley_head_kernel below), a word a thread.
// An evaluated word (its depth is at least r) is head . tail, the tail being the
// last r symbols, as the head kernel forms it.  Every regular word of length r is a
// candidate tail: a table in LDS holds their points (the maps of the tail
// applied right to left to the seed, FP64 homogeneous) in lexicographic order.
// The word's value is its head's product (FP64, left to right) at its tail's
// point.  A render's shorter words are walked right to left in full.
template <int MODE>
__global__ __launch_bounds__(256) void cayley_kernel(const CayleyJob a) {
    __shared__ uint64_t C[KL_MAX_DEPTH + 1][kCayleyMaxStates];
    __shared__ uint64_t CM[KL_MAX_DEPTH + 1][kCayleyMaxSets];
    __shared__ uint8_t NX[kCayleyMaxSets * kCayleyMaxSymbols];
    __shared__ uint16_t SETS[kCayleyMaxSets];
    __shared__ m64 G[kCayleyMaxSymbols];
    constexpr bool kTails = MODE == kCayleyEval;
    __shared__ c64 TU[kTails ? kCayleyHeadTails : 1], TV[kTails ? kCayleyHeadTails : 1];
    __shared__ uint8_t TB[kCayleyMaxStates * (kCayleyMaxSymbols + 1)];
    __shared__ uint8_t A[kCayleyMaxStates * kCayleyMaxStates];
    __shared__ uint64_t DS[KL_MAX_DEPTH + 2];
    const int S = a.S, m = a.m, M = a.n_sets, D = a.max_depth;
    const int r = kTails ? a.r : 0;
    for (int i = threadIdx.x; i < M * m; i += blockDim.x) NX[i] = a.next_set[i];
    for (int i = threadIdx.x; i < M; i += blockDim.x) SETS[i] = a.sets[i];
    for (int i = threadIdx.x; i < m; i += blockDim.x) G[i] = a.maps[i];
    for (int i = threadIdx.x; i < S * (m + 1); i += blockDim.x) TB[i] = a.table[i];
    for (int i = threadIdx.x; i < KL_MAX_DEPTH + 2; i += blockDim.x) DS[i] = a.depth_start[i];
    __syncthreads();
    cayley_counts(TB, A, &C[0][0], kCayleyMaxStates, S, m, D);
    for (int i = threadIdx.x; i < (D + 1) * M; i += blockDim.x) {
        const int L = i / M, g = i - L * M;
        uint64_t n = 0;
        for (int s = 0; s < S; ++s)
            if ((SETS[g] >> s) & 1u) n += C[L][s];
        CM[L][g] = n;
    }
    __syncthreads();

    // Unrank word `local` of length d (lexicographic, first symbol most
    // significant); symbol j chosen among the candidates by the counts of
    // their completions.  Mh becomes the product of the first hl symbols.
    auto unrank = [&](uint64_t local, int d, int hl, uint64_t& lo, uint64_t& hi, m64& Mh, uint64_t k) {
        int g = 0;
        lo = hi = 0;
        for (int j = 0; j < d; ++j) {
            const uint64_t* row = CM[d - j - 1];
            int x = 1, gx = 0;
            for (; x <= m; ++x) {
                gx = NX[g * m + x - 1];
                const uint64_t n = row[gx];
                if (local < n) break;
                local -= n;
            }
            g = gx;
            if (MODE == kCayleyDecode) a.symbols_out[k * (uint64_t)d + j] = (uint8_t)x;
            else if (j < 21) lo |= (uint64_t)(x - 1) << (3 * j);
            else hi |= (uint64_t)(x - 1) << (3 * (j - 21));
            if (j < hl) Mh = mmul(Mh, G[x - 1]);
        }
    };
    // the seed of a word whose last symbol is `last` (0-based), homogeneous
    const int seed = MODE == kCayleyRender ? a.seed_list[blockIdx.y] : a.seed;   // a render's seeds: one grid row each
    auto seed_point = [&](int last, c64& u, c64& v) {
        const int sd = seed < 0 ? last : seed;
        u = a.fix[sd];
        v = {1.0, 0.0};
        if ((a.inf_mask >> sd) & 1u) {
            u = {1.0, 0.0};
            v = {0.0, 0.0};
        }
    };
    // the maps of symbols j0 .. j1 - 1 applied right to left to (u : v)
    auto walk = [&](uint64_t lo, uint64_t hi, int j0, int j1, c64& u, c64& v) {
        for (int j = j1 - 1; j >= j0; --j) {
            const m64& Gx = G[packed_symbol(lo, hi, j)];
            const c64 nu = cfma(Gx.a, u, cmul(Gx.b, v));
            const c64 nv = cfma(Gx.c, u, cmul(Gx.d, v));
            u = nu;
            v = nv;
        }
    };

    if constexpr (kTails) {
        // the tail table: regular words of length r in lexicographic order
        for (int t = threadIdx.x; t < a.n_tails; t += blockDim.x) {
            uint64_t lo, hi;
            m64 unused;
            unrank((uint64_t)t, r, 0, lo, hi, unused, 0);
            c64 u, v;
            seed_point(packed_symbol(lo, hi, r - 1), u, v);
            walk(lo, hi, 0, r, u, v);
            cayley_tail_normalize(u, v);
            TU[t] = u;
            TV[t] = v;
        }
        __syncthreads();
    }

    uint64_t drop = 0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < a.count; k += stride) {
        int d = D;
        uint64_t local;
        if (MODE == kCayleyEval) {
            local = a.idx[k];
            if (local >= DS[1]) {
                a.z_out[k] = {__builtin_nan(""), __builtin_nan("")};
                continue;
            }
        } else {
            const uint64_t i = a.first + k;
            d = a.min_depth;
            while (i >= DS[d - a.min_depth + 1]) ++d;
            local = i - DS[d - a.min_depth];
        }
        const int hl = kTails ? d - r : 0;   // head length (r <= D = d)
        uint64_t lo, hi;
        m64 Mh = {{1.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {1.0, 0.0}};
        unrank(local, d, hl, lo, hi, Mh, k);
        if (MODE == kCayleyDecode) continue;
        double px, py;
        if constexpr (kTails) {
            // rank of the tail among the regular words of length r
            int t = 0, g = 0;
            for (int j = 0; j < r; ++j) {
                const int y = packed_symbol(lo, hi, hl + j) + 1;
                const uint64_t* row = CM[r - j - 1];
                for (int x = 1; x < y; ++x) t += (int)row[NX[g * m + x - 1]];
                g = NX[g * m + y - 1];
            }
            cayley_word(a, cayley_head(a, Mh), TU[t], TV[t], px, py);
        } else {
            c64 u, v;
            seed_point(packed_symbol(lo, hi, d - 1), u, v);
            walk(lo, hi, 0, d, u, v);
            cayley_pixel(a, u, v, px, py);
        }
        if (MODE == kCayleyEval) {
            a.z_out[k] = {px, py};
        } else {
            const uint32_t bin = cayley_bin(px, py, a.W, a.H);
            if (bin == kCayleyOutside) ++drop;
            else atomicAdd(a.image + bin, 1u);
        }
    }
    if (MODE == kCayleyRender && a.dropped) {
        for (int off = kWave / 2; off > 0; off >>= 1) drop += __shfl_down(drop, off, kWave);
        if ((threadIdx.x & (kWave - 1)) == 0 && drop) atomicAdd((unsigned long long*)a.dropped, (unsigned long long)drop);
    }
}

// ------------------------------------------------------------------ one head per thread
// Render of the words of depths >= r: a thread takes a whole head (the
// first d - r symbols) and walks the list of tails its head's good set
// accepts (built per block in LDS), so no lane re-ranks in the middle of a
// run or steps over a tail it rejects.  Heads are ranked by their own
// counts: NH[L][g] heads of L more symbols from good set g accept at least
// one tail (NH[0][g] = [CM[r][g] > 0]), so head hh of a depth unranks as a
// word does, with NH in place of CM, while the skipped CM counts give the
// index of the head's first word.  The accepted tails of a head, in table
// (lexicographic) order, are its words in index order; an index range cuts
// the first and last of its heads.  The arithmetic of a word is that of
// cayley_kernel: the head's FP64 product left to right, then cayley_pixel.
//
// The counts CM and NH satisfy the same recurrence over the good sets,
//   CM[L][g] = sum over x of CM[L - 1][next_set(g, x)],
// from CM[0][g] = [state 0 in g] and NH[0][g] = [CM[r][g] > 0], so one wave
// forms both with a lane per good set.  A thread takes a whole head, or, when
// the launch has more threads than heads, one of `parts` slices of its tails.
//
// LDS, sized from the table (HeadLayout): CM and NH rows for lengths 0..D,
// the set automaton, the tail table, and per depth the range's head offsets.
struct HeadLayout {
    // byte offsets: the job; CM, NH rows ([(D + 1) * (M + 1)], entry M of a
    // row zero); per good set its successors, a byte a symbol (NX, M for none);
    // per depth (index d - min_depth) the range's first head HA, the prefix of
    // head counts HS and the word range WA, WB; the tail points TU, TV, their
    // end states TS; and per good set g the tails it accepts, in table order,
    // at AL[g * stride]
    uint32_t job, CM, NH, NX, HA, HS, WA, WB, TU, TV, TS, AL, total;
};

// entries of a good set's tail list, padded to whole groups of kCayleyGroup
constexpr int kCayleyGroup = 4;
__host__ __device__ inline int cayley_list_stride(int n_tails) {
    return (n_tails + kCayleyGroup - 1) / kCayleyGroup * kCayleyGroup;
}

__host__ __device__ inline HeadLayout cayley_head_layout(int M, int D, int n_tails, int n_seeds) {
    HeadLayout L;
    uint32_t off = 0;
    auto take = [&](uint32_t bytes) {
        const uint32_t at = off;
        off = (off + bytes + 15u) & ~15u;
        return at;
    };
    const uint32_t rows = (uint32_t)(D + 1);
    L.job = take((uint32_t)sizeof(CayleyJob));
    L.CM = take(rows * (uint32_t)(M + 1) * 8u);
    L.NH = take(rows * (uint32_t)(M + 1) * 8u);
    L.NX = take((uint32_t)M * 8u);
    L.HA = take((KL_MAX_DEPTH + 1) * 8u);
    L.HS = take((KL_MAX_DEPTH + 2) * 8u);
    L.WA = take((KL_MAX_DEPTH + 1) * 8u);
    L.WB = take((KL_MAX_DEPTH + 1) * 8u);
    L.TU = take((uint32_t)n_seeds * (uint32_t)n_tails * (uint32_t)sizeof(c64));
    L.TV = take((uint32_t)n_seeds * (uint32_t)n_tails * (uint32_t)sizeof(c64));
    L.TS = take((uint32_t)n_tails);
    L.AL = take((uint32_t)M * (uint32_t)cayley_list_stride(n_tails) * 2u);
    L.total = off;
    return L;
}

// The symbol (x, 0-based) of rank `local` among the successors nx of a good
// set, symbol x leading to n[nx byte x] words: local becomes the rank within
// that symbol's words, g its good set, and `skipped` grows by the `also`
// counts of the symbols before it.  All counts are read together; bytes past
// the last symbol name an entry that is zero.
template <bool ALSO>
__device__ __forceinline__ void choose_symbol(const uint64_t* n, const uint64_t* also, uint64_t nx, bool wide,
                                              uint64_t& local, int& x, int& g, uint64_t& skipped) {
    uint64_t cum = 0, below = 0, cum2 = 0, below2 = 0;
    x = 0;
    auto four = [&](int y0) {
        uint64_t c[4], c2[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const int to = (int)((nx >> (8 * (y0 + y))) & 255u);
            c[y] = n[to];
            if (ALSO) c2[y] = also[to];
        }
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            cum += c[y];
            const bool past = local >= cum;
            x += past ? 1 : 0;
            below = past ? cum : below;
            if (ALSO) {
                cum2 += c2[y];
                below2 = past ? cum2 : below2;
            }
        }
    };
    four(0);
    if (wide) four(4);
    local -= below;
    if (ALSO) skipped += below2;
    g = (int)((nx >> (8 * x)) & 255u);
}

// Workgroup of the head kernel: 512 threads, two workgroups a CU, 16 waves a
// CU to hide the latency of the FP64 head products and LDS reads; every
// workgroup builds the tables above in LDS.
//
// What bounds it: at depth 16 of the once-punctured torus table (57.4 M
// words) two thirds of its 36 instructions a wave-word are the words' FP64
// ones, one third the heads' ranking and products, whose LDS reads and long
// chains leave waves waiting a third of their time (half of the issue slots
// are used: 16 waves a CU do not hide them); at shallow depths the
// chain of dependent LDS reads that builds the tables, hence the counts by
// shuffles, the symbols' counts read together, the job copied to LDS in one
// load, and one wave a good set for the tail lists.  Table 2 at depth 16:
// 92.5 us a call, with one thread a list, counts through LDS and a range
// test per word 156.8; depth 7: 15.5 against 102; the PSL(2, Z) tiling to
// depth 38 from three seeds: 114 against 160.
constexpr unsigned kCayleyHeadBlock = 512;
constexpr uint64_t kCayleyMaxParts = 16;   // slices of a head's tails: a thread keeps some 15 words

__global__ __launch_bounds__(kCayleyHeadBlock) void cayley_head_kernel(const CayleyJob job, const int M, const int D,
                                                                       const int NT, const int NS) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t odd_slots;   // seeds with a tail that is not stored as (y : 1)
    const HeadLayout lay = cayley_head_layout(M, D, NT, NS);
    const CayleyJob& a = *(const CayleyJob*)(lds + lay.job);
    uint64_t *CM = (uint64_t*)(lds + lay.CM), *NH = (uint64_t*)(lds + lay.NH), *NX = (uint64_t*)(lds + lay.NX);
    uint64_t *HA = (uint64_t*)(lds + lay.HA), *HS = (uint64_t*)(lds + lay.HS), *WA = (uint64_t*)(lds + lay.WA),
             *WB = (uint64_t*)(lds + lay.WB);
    c64 *TU_all = (c64*)(lds + lay.TU), *TV_all = (c64*)(lds + lay.TV);
    uint8_t* TS = (uint8_t*)(lds + lay.TS);
    uint16_t* AL = (uint16_t*)(lds + lay.AL);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int M1 = M + 1, LA = cayley_list_stride(NT);
    static_assert(sizeof(CayleyJob) % 4 == 0, "copied by dwords");
    for (uint32_t i = threadIdx.x; i < sizeof(CayleyJob) / 4; i += blockDim.x)
        ((uint32_t*)(lds + lay.job))[i] = ((const uint32_t*)&job)[i];
    if (threadIdx.x == 0) odd_slots = 0;
    __syncthreads();
    const int m = a.m, r = a.r;
    const bool wide = m > 4;
    static_assert(kCayleyMaxSets <= kWave, "one lane per good set");
    if (wave == 0) {
        uint64_t nx = 0;
        for (int x = 0; x < 8; ++x) nx |= (uint64_t)(x < m && lane < M ? a.next_set[lane * m + x] : M) << (8 * x);
        if (lane < M) NX[lane] = nx;
        uint64_t cm = lane < M ? a.sets[lane] & 1u : 0u, nh = 0;
        for (int L = 0;; ++L) {
            if (L == r) nh = cm > 0 ? 1 : 0;
            if (lane <= M) {
                CM[L * M1 + lane] = cm;
                if (L >= r) NH[(L - r) * M1 + lane] = nh;
            }
            if (L == D) break;
            uint64_t c = 0, h = 0;
            auto four = [&](int y0) {
#pragma unroll
                for (int y = y0; y < y0 + 4; ++y) {
                    // a set index of M (no symbol) names lane M, or with 64 sets none
                    const int to = (int)((nx >> (8 * y)) & 255u);
                    const uint64_t cv = __shfl(cm, to & (kWave - 1), kWave), hv = __shfl(nh, to & (kWave - 1), kWave);
                    c += to < M ? cv : 0;
                    h += to < M ? hv : 0;
                }
            };
            four(0);
            if (wide) four(4);
            cm = lane < M ? c : 0;
            nh = lane < M ? h : 0;
        }
        // with 64 sets no lane holds the rows' zero entry
        if (M == kWave && lane <= D) CM[lane * M1 + M] = NH[lane * M1 + M] = 0;
    }
    __syncthreads();
    // the tail table: regular words of length r in lexicographic order, their
    // end states, and their points from each seed in turn (TU[slot * NT + t])
    for (int e = threadIdx.x; e < NS * NT; e += blockDim.x) {
        const int slot = e / NT, t = e - slot * NT;
        uint64_t local = (uint64_t)t, lo = 0, hi = 0, unused = 0;
        int g = 0;
        for (int j = 0; j < r; ++j) {
            int x;
            choose_symbol<false>(CM + (r - j - 1) * M1, nullptr, NX[g], wide, local, x, g, unused);
            if (j < 21) lo |= (uint64_t)x << (3 * j);
            else hi |= (uint64_t)x << (3 * (j - 21));
        }
        if (slot == 0) {
            int s = 0;
            for (int j = r - 1; j >= 0; --j) s = a.table[s * (m + 1) + packed_symbol(lo, hi, j) + 1];
            TS[t] = (uint8_t)s;
        }
        const int last = packed_symbol(lo, hi, r - 1);
        const int sd = a.seed_list[slot] < 0 ? last : a.seed_list[slot];
        c64 u = a.fix[sd], v = {1.0, 0.0};
        if ((a.inf_mask >> sd) & 1u) {
            u = {1.0, 0.0};
            v = {0.0, 0.0};
        }
        for (int j = r - 1; j >= 0; --j) {
            const m64& Gx = a.maps[packed_symbol(lo, hi, j)];
            const c64 nu = cfma(Gx.a, u, cmul(Gx.b, v));
            const c64 nv = cfma(Gx.c, u, cmul(Gx.d, v));
            u = nu;
            v = nv;
        }
        cayley_tail_normalize(u, v);
        TU_all[e] = u;
        TV_all[e] = v;
        if (!(v.re == 1.0 && v.im == 0.0)) atomicOr(&odd_slots, 1u << slot);
    }
    // per depth: the range's local word interval and the heads it touches
    const int d0 = r > a.min_depth ? r : a.min_depth;
    for (int e = threadIdx.x; e < 2 * (D - d0 + 1); e += blockDim.x) {
        const int d = d0 + e / 2, di = d - a.min_depth, hl = d - r;
        const uint64_t s0 = a.depth_start[di], s1 = a.depth_start[di + 1];
        const uint64_t lo_w = a.first > s0 ? a.first - s0 : 0;
        const uint64_t end = a.first + a.count;
        const uint64_t hi_w = end < s1 ? (end > s0 ? end - s0 : 0) : s1 - s0;
        if (e % 2 == 0) {
            WA[di] = lo_w;
            WB[di] = hi_w;
        }
        // rank of the head of word lo_w (e even) or hi_w - 1 (e odd): the
        // first or last of its depth where the range does not cut it
        uint64_t hr = 0;
        if (hi_w > lo_w) {
            if (e % 2 ? end >= s1 : lo_w == 0) {
                hr = e % 2 ? NH[hl * M1] - 1 : 0;
            } else {
                uint64_t local = e % 2 == 0 ? lo_w : hi_w - 1;
                int g = 0, x;
                for (int j = 0; j < hl; ++j)
                    choose_symbol<true>(CM + (d - j - 1) * M1, NH + (hl - j - 1) * M1, NX[g], wide, local, x, g, hr);
            }
        }
        if (e % 2 == 0) HA[di] = hr;
        else HS[di] = hr;   // the last head, turned into a count below
    }
    __syncthreads();
    // per good set, the tails it accepts in table order (as byte offsets of
    // their points): one wave a set, 64 tails at a time
    for (int g = wave; g < M; g += (int)(blockDim.x / kWave)) {
        const uint32_t set = a.sets[g];
        int k = 0;
        for (int t0 = 0; t0 < NT; t0 += kWave) {
            const int t = t0 + lane;
            const bool in = t < NT && ((set >> TS[t]) & 1u);
            const uint64_t b = __ballot(in);
            if (in) AL[g * LA + k + __popcll(b & ((1ull << lane) - 1))] = (uint16_t)(t * sizeof(c64));
            k += __popcll(b);
        }
    }
    if (threadIdx.x == 0) {
        uint64_t total = 0;
        for (int d = d0; d <= D; ++d) {
            const int di = d - a.min_depth;
            const uint64_t n = WB[di] > WA[di] ? HS[di] - HA[di] + 1 : 0;
            HS[di] = total;
            total += n;
        }
        HS[D - a.min_depth + 1] = total;
    }
    __syncthreads();

    // (seed, head, part) triples, seed-major so that the lanes of a wave share
    // a seed, a head's parts on neighbouring lanes
    const uint64_t total = HS[D - a.min_depth + 1];
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t heads = total * (uint64_t)NS;
    const uint32_t parts = heads ? (uint32_t)max((uint64_t)1, min(kCayleyMaxParts, stride / heads)) : 1u;
    uint64_t drop = 0;
    uint64_t run_key = kCayleyOutsideKey;
    uint32_t run_len = 0;
    const uint32_t W = job.W, H = job.H;
    uint32_t* image = job.image;   // from the argument: an address read from LDS would make flat atomics
    auto close_run = [&]() {
        const uint32_t col = (uint32_t)run_key, row = (uint32_t)(run_key >> 32);
        if ((col < W) & (row < H)) {
            if (run_len) atomicAdd(image + __umul24(row, W) + col, run_len);
        } else {
            drop += run_len;
        }
        run_len = 0;
    };
    auto emit = [&](uint64_t key) {
        if (key != run_key) {
            close_run();
            run_key = key;
        }
        ++run_len;
    };
    for (uint64_t uu = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; uu < heads * parts; uu += stride) {
        const uint64_t hu = parts == 1 ? uu : uu / parts;
        const uint32_t part = (uint32_t)(uu - hu * parts);
        const int slot = hu < total ? 0 : (int)(hu / total);
        const uint64_t u = hu - (uint64_t)slot * total;
        const unsigned char* TU = (const unsigned char*)(TU_all + (size_t)slot * NT);
        const unsigned char* TV = (const unsigned char*)(TV_all + (size_t)slot * NT);
        int d = d0;
        while (u >= HS[d + 1 - a.min_depth]) ++d;
        const int di = d - a.min_depth, hl = d - r;
        uint64_t hh = HA[di] + (u - HS[di]);
        // unrank the head by NH; the skipped CM counts give its first word
        int g = 0;
        uint64_t wstart = 0;
        m64 Mh = {{1.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {1.0, 0.0}};
        for (int j = 0; j < hl; ++j) {
            int x;
            choose_symbol<true>(NH + (hl - j - 1) * M1, CM + (d - j - 1) * M1, NX[g], wide, hh, x, g, wstart);
            Mh = mmul(Mh, a.maps[x]);
        }
        // this head's accepted tails with ordinals in [o0, o1) are words of the
        // range, this part's share of them (whole groups)
        const uint64_t wa = WA[di], wb = WB[di], n_acc = CM[r * M1 + g];
        uint32_t o0 = (uint32_t)(wa > wstart ? wa - wstart : 0);
        uint32_t o1 = (uint32_t)(wb - wstart < n_acc ? wb - wstart : n_acc);
        if (parts > 1) {
            const uint32_t per = (uint32_t)((n_acc + kCayleyGroup * parts - 1) / (kCayleyGroup * parts)) * kCayleyGroup;
            o0 = max(o0, part * per);
            o1 = min(o1, (part + 1) * per);
        }
        const uint16_t* list = AL + (size_t)g * LA;
        const CayleyHead ch = cayley_head(a, Mh);
        uint32_t i = o0;
        if (ch.pole && !((odd_slots >> slot) & 1u)) {
            // every tail is (y : 1): groups of kCayleyGroup tails, their list
            // entries in one read and their points read before use
            auto one = [&](uint32_t off) {
                double px, py;
                cayley_pole_word(ch, *(const c64*)(TU + off), px, py);
                emit(cayley_pole_key(px, py));
            };
            for (; i < o1 && (i & (kCayleyGroup - 1)); ++i) one(list[i]);
            for (; i + kCayleyGroup <= o1; i += kCayleyGroup) {
                const uint2 w = *(const uint2*)(list + i);
                const uint32_t off[kCayleyGroup] = {w.x & 0xFFFFu, w.x >> 16, w.y & 0xFFFFu, w.y >> 16};
                c64 y[kCayleyGroup];
                uint64_t key[kCayleyGroup];
#pragma unroll
                for (int e = 0; e < kCayleyGroup; ++e) y[e] = *(const c64*)(TU + off[e]);
#pragma unroll
                for (int e = 0; e < kCayleyGroup; ++e) {
                    double px, py;
                    cayley_pole_word(ch, y[e], px, py);
                    key[e] = cayley_pole_key(px, py);
                }
#pragma unroll
                for (int e = 0; e < kCayleyGroup; ++e) emit(key[e]);
            }
            for (; i < o1; ++i) one(list[i]);
        } else {
            for (; i < o1; ++i) {
                const uint32_t off = list[i];
                double px, py;
                cayley_word(a, ch, *(const c64*)(TU + off), *(const c64*)(TV + off), px, py);
                const bool number = (px == px) & (py == py);
                emit(number ? cayley_pole_key(px, py) : kCayleyOutsideKey);
            }
        }
    }
    close_run();
    if (job.dropped) {
        for (int off = kWave / 2; off > 0; off >>= 1) drop += __shfl_down(drop, off, kWave);
        if (lane == 0 && drop) atomicAdd((unsigned long long*)job.dropped, (unsigned long long)drop);
    }
}

hipError_t launch_cayley(const CayleyJob& job, int mode, hipStream_t s) {
    if (job.count == 0) return hipSuccess;
    CayleyJob j = job;
    const unsigned grid = (unsigned)std::max(1, j.grid_blocks);
    if (mode == kCayleyRender) {
        // words of depths >= r go one head per thread
        const uint64_t B = j.r > j.min_depth ? j.depth_start[j.r - j.min_depth] : 0;   // first word of depth r
        const uint64_t end = j.first + j.count;
        if (end > B) {
            CayleyJob h = j;
            h.first = j.first > B ? j.first : B;
            h.count = end - h.first;
            // as many seeds per launch as their tail tables fit the LDS of a CU
            const size_t cap = 160 * 1024 - 16;   // less the kernel's static LDS
            int per = j.n_seeds;
            while (per > 1 && cayley_head_layout(j.n_sets, j.max_depth, j.n_tails, per).total > cap) --per;
            for (int k0 = 0; k0 < j.n_seeds; k0 += per) {
                h.n_seeds = std::min(per, j.n_seeds - k0);
                for (int k = 0; k < h.n_seeds; ++k) h.seed_list[k] = j.seed_list[k0 + k];
                const size_t lds = cayley_head_layout(j.n_sets, j.max_depth, j.n_tails, h.n_seeds).total;
                if (lds > 65536) {
                    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(cayley_head_kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                    if (e != hipSuccess) return e;
                }
                hipLaunchKernelGGL(cayley_head_kernel, dim3(grid), dim3(kCayleyHeadBlock), lds, s, h, h.n_sets, h.max_depth,
                                   h.n_tails, h.n_seeds);
                hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
            }
        }
        if (j.first >= B) return hipSuccess;
        j.count = std::min(end, B) - j.first;   // the words shorter than r
    }
    const unsigned blocks = (unsigned)std::min<uint64_t>((j.count + 255) / 256, grid);
    if (mode == kCayleyDecode) hipLaunchKernelGGL(cayley_kernel<kCayleyDecode>, dim3(blocks), dim3(256), 0, s, j);
    else if (mode == kCayleyEval) hipLaunchKernelGGL(cayley_kernel<kCayleyEval>, dim3(blocks), dim3(256), 0, s, j);
    else hipLaunchKernelGGL(cayley_kernel<kCayleyRender>, dim3(blocks, (unsigned)j.n_seeds), dim3(256), 0, s, j);
    return hipGetLastError();
}

}  // namespace kl
