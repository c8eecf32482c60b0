// host_rules.hpp -- decisions of the host side that need no device, in plain
// C++ so that they can be compiled and checked by themselves.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace kl {

// ------------------------------------------------------------------ device buffer
// Each device keeps one buffer for the tables and staged points of calls on
// the null stream (Temp::tables in abi.cpp).  Largest buffer it holds, and the
// size above which it is given back after kTableCacheIdle calls in a row
// that a buffer of that size would have served.  A walk render of 2^26 points
// takes 152 MB, a batch of 256 sets of depths 12..18 some 110: mapped and
// unmapped on each call, as the stream-ordered allocator does around a
// synchronisation, they cost 420 and 400 us beside 200 us and 9.9 ms of kernels.
constexpr size_t kTableCacheMax = size_t(192) << 20, kTableCacheKeep = size_t(64) << 20,
                 kTableCacheMin = size_t(1) << 20;
constexpr int kTableCacheIdle = 32;

struct TableLease {
    bool lease;      // the call uses the buffer
    bool release;    // the buffer held so far is freed first
    size_t allocate; // then one of this size is allocated (0: none)
};

// A call that asks for `want` bytes while `held` are held (0: none) and no
// other call uses them; `idle` counts the calls in a row that
// kTableCacheKeep bytes would have served, or that no buffer would have: a
// call above kTableCacheMax takes a temporary, and so does not use one either.
inline TableLease table_lease(size_t held, size_t want, int& idle) {
    const bool fits = want <= kTableCacheMax;
    idle = fits && want > kTableCacheKeep ? 0 : std::min(idle + 1, kTableCacheIdle);
    const bool tired = held > kTableCacheKeep && idle == kTableCacheIdle;
    if (!fits) return {false, tired, 0};
    if (held < want || tired) return {true, held > 0, std::max(want, kTableCacheMin)};
    return {true, false, 0};
}

// ------------------------------------------------------------------ batched renders
// Whether a batched render whose longest suffixes have `letters` letters adds
// up its runs by bin in LDS first (kernels.hip, MergeSink); `bins` an image,
// `tiling` all sets into one, `units` of 256 heads in all.  A run then waits for the table where a global
// atomic would not be waited for, and fewer atomics leave the chip.  With
// six letters runs are long and few: 60 sets of depths 9 .. 13 231 us merged
// and 150 not, ten of depths 11 .. 13 110 and 97.  With five, FP32 (five
// waves a SIMD) gains where the atomics are many: Maskit's tilings to depth 15
// at 300^2 / 1024^2 / 4096^2 137 / 148 / 294 us merged and 158 / 201 / 377 not,
// two sets of depth 17 172 and 252, though sets of few units lose up to a
// fifth (40 of depths 11 .. 13 at 1024^2 116 and 92).  FP64 (three waves) has
// less to run while it waits: the tilings to depth 16 at 512^2 / 1024^2 /
// 2048^2 432 / 467 / 495 us merged and 377 / 392 / 452 not, to depth 15 at
// 512^2 198 and 176, forty sets 144 and 110; only images that exceed the caches
// favour merging (2900^2 / 4096^2 / 8192^2, depth 16: 510 / 527 / 663 and
// 530 / 622 / 927; depth 15: 242 / 294 / 478 and 325 / 393 / 558), so it is kept
// for those of 2^23 bins up, where units are few (5,500 at depth 16; depth 18,
// five letters, 12,400 units: at 4096^2 849 and 771).  With four and fewer letters both gain: depth 14
// 100 and 138 us, in FP64 106 and 136.
inline bool batch_merges(bool fp64, int letters, bool tiling, uint64_t bins, uint64_t units) {
    return letters <= 4 || (letters == 5 && (!fp64 || (tiling && bins >= (uint64_t(1) << 23) && units < 8192)));
}

}  // namespace kl
