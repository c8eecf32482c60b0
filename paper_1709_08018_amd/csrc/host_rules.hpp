// host_rules.hpp -- decisions of the host side that need no device, in plain
// C++ so that they can be compiled and checked by themselves.
#pragma once

#include <stddef.h>

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

}  // namespace kl
