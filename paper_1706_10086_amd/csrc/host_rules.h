// Rules of the host side that need no GPU, in plain C++: tests compile this file alone
// and check the rules on the CPU.
#pragma once

#include <stdint.h>

namespace mgemm {

// Whether `blocks` work-groups of `threads` threads fit one dimension of a grid: a
// launch counts work-items in 32 bits (a dispatch beyond that would run part of them).
inline bool grid_fits(int64_t blocks, int64_t threads) { return blocks <= 0xFFFFFFFFll / threads; }

// Work-groups of the direct-load kernels that share launches or a plan.
constexpr int64_t DIRECT_THREADS = 256;
// Products of one shared launch at most (their descriptions stay below 4 KiB of kernel
// arguments).
constexpr int LIST_MAX = 56;

// Whether LIST_MAX products of m x n may share a launch on the smallest tile.
inline bool list_grid_fits(int64_t m, int64_t n) {
    const int64_t tiles = ((m + 31) / 32) * ((n + 31) / 32);
    return grid_fits(tiles * LIST_MAX, DIRECT_THREADS);
}

}  // namespace mgemm
