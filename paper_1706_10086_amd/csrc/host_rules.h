// Rules of the host side that need no GPU, in plain C++: tests compile this file alone
// and check the rules on the CPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

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

// ---------------------------------------------------------------------------
// Lists whose products share launches.
// ---------------------------------------------------------------------------
// Bytes that a product of a list reads or writes.
struct Span {
    uintptr_t b, e;
    bool write;
};

inline void add_span(std::vector<Span> &v, const void *p, int64_t r, int64_t c, int64_t ld, size_t es,
                     bool write) {
    v.push_back({(uintptr_t)p, (uintptr_t)p + (size_t)((r - 1) * ld + c) * es, write});
}

// Whether a written span meets any other span.
inline bool written_twice_or_read(std::vector<Span> &v) {
    std::sort(v.begin(), v.end(), [](const Span &x, const Span &y) { return x.b < y.b; });
    uintptr_t any_end = 0, write_end = 0;        // furthest ends so far
    for (const Span &s : v) {
        if (s.b < (s.write ? any_end : write_end)) return true;
        any_end = std::max(any_end, s.e);
        if (s.write) write_end = std::max(write_end, s.e);
    }
    return false;
}

// Runs products [i0, i1) of a list, which do not depend on each other: run(i, &joins)
// runs product i or sets joins, and the products that joined run together at the end.
// Where one fails, those before it -- the joined ones too -- still run, as in a list
// run in turn; failed() is called before them, for the error's message.
template <typename Run, typename RunGroup, typename Failed>
int32_t run_window(int64_t i0, int64_t i1, Run run, RunGroup run_group, Failed failed) {
    std::vector<int64_t> group;
    int32_t rc = 0;
    for (int64_t i = i0; i < i1 && rc == 0; ++i) {
        bool joins = false;
        rc = run(i, &joins);
        if (rc == 0 && joins) group.push_back(i);
    }
    if (rc) failed();
    if (!group.empty()) {
        const int32_t grc = run_group(group);
        if (rc == 0) rc = grc;
    }
    return rc;
}

// ---------------------------------------------------------------------------
// Which networks train on the step kernel.
// ---------------------------------------------------------------------------
constexpr int STEP_MAX_IN = 32, STEP_MAX_HIDDEN = 128;

// Training rows per tile of the step kernel.
inline int step_rows(int hidden) { return hidden <= 64 ? 64 : 32; }

// Work-groups of the step kernel for a network and a training set (at most one per
// compute unit): 0 where the step runs layer by layer instead.
//
// A work-group takes the outputs 64 at a time, and the layer-by-layer path spreads them
// over the GPU, so of many outputs the step kernel needs many rows: a step of 64 hidden
// units on 64 rows takes 42 us against 74 layer by layer with 247 outputs, 108 against
// 108 with 1024, 381 against 249 with 4096 (with 13600 rows 459 against 864).  Above 64
// hidden units a work-group that takes a second tile of 32 rows reads and rewrites its
// whole gradient share, which costs as much as it saves once rounds x outputs passes
// about 4000: 128 hidden units, 13600 rows (two rounds) 124 against 233 us with 247
// outputs, 318 against 396 with 1024, 665 against 630 with 2048; 60000 rows (eight) 470
// against 557 with 247, 766 against 754 with 512, 1349 against 1252 with 1024.
inline int step_blocks(int in, int hidden, int out, int64_t rows, int cus) {
    if (in > STEP_MAX_IN || hidden > STEP_MAX_HIDDEN || cus < 1) return 0;
    const int64_t tiles = (rows + step_rows(hidden) - 1) / step_rows(hidden);
    if (out > 768 && rows < out) return 0;
    if (hidden > 64 && (tiles + cus - 1) / cus * out > 2048) return 0;
    return (int)std::min<int64_t>(tiles, cus);
}

}  // namespace mgemm
