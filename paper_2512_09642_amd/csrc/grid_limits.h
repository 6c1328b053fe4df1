// What one launch may hold (host code without HIP dependency).
#pragma once

#include <cstdint>

namespace sstep {

// HIP refuses a launch of 2^32 threads or more.
inline bool launch_fits(uint64_t blocks, uint32_t threads) { return blocks * threads < (uint64_t(1) << 32); }

// Blocks of a launch that goes in several: of at most 1024 threads, they fit.
constexpr uint32_t kBlocksPerLaunch = uint32_t(1) << 21;

// f(first block, blocks) for each launch of a grid of any number of blocks; the
// first failure ends it.
template <class E, class F>
inline E in_launches(uint64_t blocks, E ok, F &&f)
{
    E e = ok;
    for (uint64_t first = 0; first < blocks && e == ok; first += kBlocksPerLaunch) {
        const uint64_t left = blocks - first;
        e = f(first, static_cast<uint32_t>(left < kBlocksPerLaunch ? left : kBlocksPerLaunch));
    }
    return e;
}

}  // namespace sstep
