// walk_layout.hpp -- host-side sizes of the binned walk render (walk.hip):
// which images and walks it takes, and how its staging is laid out.  Plain
// C++ with no device code.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace kl {

constexpr uint32_t kWalkTileBits = 15;                    // a tile: 2^15 bins
constexpr uint32_t kWalkTileBins = 1u << kWalkTileBits;
constexpr uint32_t kMaxWalkTiles = 256;
// A region holds a workgroup's drawn points of one Philox block, eight steps
// at most, so that a step's place in its region is known at compile time and
// its bin and rank stay in registers.  (Sixteen steps a region took 15%
// longer on 2^30 points, thirty-two 72% longer, and four no shorter.)
constexpr uint32_t kWalkChunk = 8;
// Walkers of a workgroup, and those of a workgroup whose regions would not
// fit the staging otherwise (walk_binned_layout).
constexpr uint32_t kWalkBlock = 512, kWalkBlockSmall = 256;
// Longest binned walk, and the slots (2 bytes each) of the regions that one
// launch stages at most: those of a small workgroup of the longest walks,
// whose drawn steps 1 .. 2^19 touch 2^16 + 1 blocks of eight.
constexpr uint32_t kWalkBinnedSteps = 1u << 19;
constexpr uint64_t kWalkBinnedSlots = (uint64_t)kWalkBlockSmall * kWalkChunk * (kWalkBinnedSteps / kWalkChunk + 1);

inline uint32_t walk_tiles(uint32_t W, uint32_t H) {
    const uint64_t bins = (uint64_t)W * H;
    return (uint32_t)((bins + kWalkTileBins - 1) / kWalkTileBins);
}

// The binned render takes the image and the walk.
inline bool walk_binned_ok(uint32_t W, uint32_t H, uint32_t n_steps) {
    return walk_tiles(W, H) <= kMaxWalkTiles && n_steps <= kWalkBinnedSteps;
}

// Regions of a workgroup: the Philox blocks with a drawn step
// burn_in + 1 .. burn_in + n_steps, n_steps >= 1.
inline uint32_t walk_chunks(uint32_t burn_in, uint32_t n_steps) {
    return (burn_in + n_steps) / kWalkChunk - (burn_in + 1) / kWalkChunk + 1;
}

// The temporaries of a binned render (walk_binned_ok): `blocks` workgroups of
// `walkers` walkers a launch, their regions' slots (walkers * kWalkChunk a
// region, at most kWalkBinnedSlots) from the start on, and from off_starts on
// each region's tile starts (one a tile, and their end).
struct WalkBinned {
    uint32_t walkers, chunks;
    uint64_t blocks;           // 0: nothing to draw
    size_t off_starts, bytes;
};

inline WalkBinned walk_binned_layout(uint64_t n_walkers, uint32_t burn_in, uint32_t n_steps, uint32_t tiles) {
    WalkBinned L{};
    if (n_walkers == 0 || n_steps == 0) return L;
    L.chunks = walk_chunks(burn_in, n_steps);
    // some 2^18 steps and more: a workgroup of 512 alone would exceed the
    // staging; 256 walkers never do
    L.walkers = (uint64_t)kWalkBlock * kWalkChunk * L.chunks <= kWalkBinnedSlots ? kWalkBlock : kWalkBlockSmall;
    const uint64_t slots = (uint64_t)L.walkers * kWalkChunk * L.chunks;   // of a workgroup
    L.blocks = std::min((n_walkers + L.walkers - 1) / L.walkers, kWalkBinnedSlots / slots);
    L.off_starts = L.blocks * slots * sizeof(uint16_t);
    L.bytes = L.off_starts + L.blocks * L.chunks * (size_t)(tiles + 1) * sizeof(uint32_t);
    return L;
}

// Whether the first launch of walkers also clears the image of `bins` bins,
// or a launch of its own does: up to 128 bins a thread of the walkers.  The
// walkers' workgroups clear some 100 GB/s each before they step, a launch of
// its own the whole image at the device's rate for some 2 us and a gap.  64
// steps, with the clearing launch and fused: 1024^2 from 16 workgroups (128
// bins a thread) 53.2 and 52.7 us, from 8 52.7 and 53.9, from one 50.0 and
// 76.7; 2048^2 from 64 workgroups (128) 65.1 and 63.7, from 32 62.8 and 63.4,
// from 4 57.6 and 83.0; 2890^2 from 512 (32) 119.4 and 114.6, from 64 (255)
// 79.9 and 78.6, from 16 75.5 and 84.4, from one 64.4 and 278.
inline bool walk_clears(const WalkBinned& L, uint64_t bins) { return bins <= 128 * L.blocks * L.walkers; }

}  // namespace kl
