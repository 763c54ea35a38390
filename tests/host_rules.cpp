// C entry points of the host rules (csrc/host_rules.h) for tests/test_host_rules.py.
#include "host_rules.h"

using namespace mgemm;

extern "C" {

int grid_fits_c(int64_t blocks, int64_t threads) { return grid_fits(blocks, threads); }

int may_hold_c(int64_t have, int64_t free, int64_t need) { return may_hold(have, free, need); }

int direct_loads_c(int64_t es, int64_t bm, int64_t bn, int64_t bk, int64_t m, int64_t n, int64_t k,
                   int64_t A, int64_t lda, int64_t B, int64_t ldb) {
    return direct_loads(es, bm, bn, bk, m, n, k, (const void *)A, lda, (const void *)B, ldb);
}

int list_joins_c(int64_t es, int64_t m, int64_t n, int64_t k, int64_t A, int64_t lda, int64_t B,
                 int64_t ldb, int64_t ldc) {
    return list_joins(es, m, n, k, (const void *)A, lda, (const void *)B, ldb, ldc);
}

int list_grid_fits_c(int64_t m, int64_t n) { return list_grid_fits(m, n); }

double tile_time_c(int f32, int tile, int64_t m, int64_t n, int64_t k, int64_t S, int64_t kc, int cus) {
    return tile_time((f32 ? kTileCostsF32 : kTileCostsF64)[tile], m, n, k, S, kc, cus);
}

int tile_taken_c(int f32, int tile, int64_t m, int64_t n, int64_t k, int64_t S, int cus) {
    return tile_taken((f32 ? kTileCostsF32 : kTileCostsF64)[tile], m, n, k, S, cus);
}

void tile_c(int f32, int tile, int32_t *bm, int32_t *bn, int32_t *bk) {
    const TileCost &d = (f32 ? kTileCostsF32 : kTileCostsF64)[tile];
    *bm = d.bm;
    *bn = d.bn;
    *bk = d.bk;
}

int step_blocks_c(int in, int hidden, int out, int64_t rows, int cus) {
    return step_blocks(in, hidden, out, rows, cus);
}

// Spans [b, e) of a list, each with a flag for written ones.
int dependent_c(int count, const int64_t *b, const int64_t *e, const int32_t *write) {
    std::vector<Span> v;
    for (int i = 0; i < count; ++i)
        add_span(v, (const void *)(uintptr_t)b[i], 1, e[i] - b[i], e[i] - b[i], 1, write[i] != 0);
    return written_twice_or_read(v);
}

// Products 0..count-1 with what they do (0: run alone, 1: join, < 0: fail with that
// code); `order` receives them as they run, `*told` how many had run when the failure
// was told.  group_rc: what the joined products' launch returns.
int window_c(int count, const int32_t *what, int group_rc, int32_t *order, int *ran, int *told) {
    *ran = 0;
    *told = -1;
    return run_window(
        0, count,
        [&](int64_t i, bool *joins) -> int32_t {
            if (what[i] < 0) return what[i];
            *joins = what[i] == 1;
            if (!*joins) order[(*ran)++] = (int32_t)i;
            return 0;
        },
        [&](const std::vector<int64_t> &g) -> int32_t {
            for (int64_t i : g) order[(*ran)++] = (int32_t)i;
            return group_rc;
        },
        [&] { *told = *ran; });
}

}  // extern "C"
