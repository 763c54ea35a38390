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

// Whether the direct-load tiles of BM x BN x BK take a product's operands (es: bytes of an
// element): at least one 16-byte unit per row of A and B, bases on 4-byte boundaries
// (the direct loads take any such address) and panels that 32-bit byte offsets span.
inline bool direct_loads(int64_t es, int64_t bm, int64_t bn, int64_t bk, int64_t m, int64_t n, int64_t k,
                         const void *A, int64_t lda, const void *B, int64_t ldb) {
    const int64_t lim = (int64_t)1 << 31;
    return m >= 1 && k >= 1 && n >= 16 / es && ((uintptr_t)A % 4) == 0 && ((uintptr_t)B % 4) == 0 &&
           bm * lda * es < lim && (bk * ldb + bn) * es < lim;
}

// Products of one shared launch at most (their descriptions stay below 4 KiB of kernel
// arguments).
constexpr int LIST_MAX = 56;
// Beyond this (tens of microseconds alone) a product gains nothing from company and takes
// its own tile.
constexpr double LIST_FLOPS = 4e9;

// Whether LIST_MAX products of m x n may share a launch on the smallest tile.
inline bool list_grid_fits(int64_t m, int64_t n) {
    const int64_t tiles = ((m + 31) / 32) * ((n + 31) / 32);
    return grid_fits(tiles * LIST_MAX, DIRECT_THREADS);
}

// Whether a product may share a launch: operands, rows and work-items in 32 bits on every
// tile of the table.
inline bool list_joins(int64_t es, int64_t m, int64_t n, int64_t k, const void *A, int64_t lda,
                       const void *B, int64_t ldb, int64_t ldc) {
    const int64_t lim = (int64_t)1 << 31;
    return direct_loads(es, 128, 128, 64, m, n, k, A, lda, B, ldb) && m < lim && k < lim && ldc < lim &&
           2.0 * (double)m * (double)n * (double)k <= LIST_FLOPS && list_grid_fits(m, n);
}

// Whether a buffer of `have` bytes holds `need`, or one of `need` bytes fits the free
// memory once it is given back.
inline bool may_hold(size_t have, size_t free, size_t need) { return have >= need || have + free >= need; }

// ---------------------------------------------------------------------------
// The direct-load tiles and their times.
// ---------------------------------------------------------------------------
// A tile and its time: with q = ceil(tiles / CUs) work-groups for the busiest
// compute unit, R of them at a time, and k rounded up to the k-step,
//   t = start + each q + rate k (BM BN / 4096) (sum over rounds of (alone + r))
// microseconds, r work-groups in the round (R in all but the last): `alone` is the
// part of a k-step that co-resident work-groups hide from each other, `each` a
// tile's prologue and epilogue.  The coefficients are least squares on the log
// of the times of 119 shapes per type (squares 64-8192, log-uniform 32-8192 and large
// ragged ones, MI355X, calls back to back, within 4-13 % rms); picking by them
// reaches 0.991 of the best tile of each shape in both types (geometric mean).
struct TileCost {
    int bm, bn, bk;
    int resident;            // R: work-groups a compute unit holds (LDS, registers)
    double start, each, rate, alone;
};

constexpr int DIRECT_TILES = 6;

constexpr TileCost kTileCostsF64[DIRECT_TILES] = {
    {128, 128, 16, 2, 0.00, 9.90, 0.02724, 0.081}, {64, 128, 16, 3, 2.16, 4.29, 0.02675, 0.278},
    {64, 64, 16, 4, 2.98, 1.96, 0.02792, 0.369},   {64, 32, 16, 5, 2.49, 1.19, 0.02768, 1.000},
    {32, 32, 32, 4, 2.58, 0.89, 0.02839, 0.874},   {32, 32, 16, 8, 2.36, 0.63, 0.03099, 1.465},
};

constexpr TileCost kTileCostsF32[DIRECT_TILES] = {
    {128, 128, 32, 2, 3.90, 6.90, 0.01490, 0.038}, {64, 128, 32, 3, 4.12, 2.53, 0.01463, 0.150},
    {64, 64, 32, 4, 3.94, 1.35, 0.01475, 0.349},   {64, 32, 32, 5, 3.59, 0.87, 0.01520, 0.643},
    {32, 32, 64, 4, 3.23, 0.83, 0.01503, 0.879},   {32, 32, 32, 8, 3.03, 0.50, 0.01706, 0.995},
};

inline int64_t tiles_of(const TileCost &d, int64_t m, int64_t n) {
    return ((m + d.bm - 1) / d.bm) * ((n + d.bn - 1) / d.bn);
}

// The time of S ranges of kc values of k each, the last one holding what is left of k (S
// = 1 and kc = k: a product run whole).  The work-groups of a shorter last range start
// last and count as the part f of a full one that they are: they go to the compute units
// that the full ones leave a work-group short, as many as fit, and then to all in turn.
// (Counted as full ones, the tiles that leave units short looked best: of 122 products
// whose k is cut for 128 x 128 tiles the pick reached 0.959 of the best tile's time,
// 0.983 with f; FP32 1441 x 488 x 5140, five ranges of which the last holds 20 values,
// 99 and 80 us.)
inline double tile_time(const TileCost &d, int64_t m, int64_t n, int64_t k, int64_t S, int64_t kc,
                        int cus) {
    const int64_t t = tiles_of(d, m, n);
    auto whole_steps = [&](int64_t v) { return (double)((v + d.bk - 1) / d.bk * d.bk); };
    const double ks = whole_steps(kc), f = whole_steps(k - (S - 1) * kc) / ks;
    const int64_t full = f < 1.0 ? t * (S - 1) : t * S, part = t * S - full;
    double busiest = (double)((full + cus - 1) / cus);          // full work-groups
    const int64_t gaps = full % cus ? (cus - full % cus) * (int64_t)(1.0 / f) : 0;
    if (part > gaps) busiest += (double)((part - gaps + cus - 1) / cus) * f;
    const double q = (double)((t * S + cus - 1) / cus);
    const double rounds = (double)(int64_t)(busiest / d.resident), last = busiest - rounds * d.resident;
    const double shared = rounds * (d.alone + d.resident) + (last > 0 ? d.alone + last : 0.0);
    return d.start + d.each * q + d.rate * ks * (d.bm * d.bn / 4096.0) * shared;
}

// Whether a product may run on the tile.  The coefficients, fitted to longer products,
// make the 128-wide tiles of a short product look better than they are where all of its
// 64 x 64 tiles are resident at once: of 16 such products with k up to 512 that the
// estimate gave to a 128-wide tile none ran faster there (1.03-1.37x as fast on the best
// of the others: FP64 722 x 4414 x 32 13.7 and 11.6 us, FP32 1330 x 1468 x 27 11.2 and
// 8.6).  With k = 2048 the 128-wide tiles win (FP32 2048 x 2048: 133 and 138).
inline bool tile_taken(const TileCost &d, int64_t m, int64_t n, int64_t k, int64_t S, int cus) {
    const TileCost square = {64, 64, 0, 4, 0, 0, 0, 0};
    return !(S == 1 && k <= 512 && d.bn >= 128 && tiles_of(square, m, n) <= (int64_t)square.resident * cus);
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
