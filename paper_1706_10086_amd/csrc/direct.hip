// The kernels behind the built-in choice: direct-load tiles (pipe_gemm.h) of six
// sizes per type, for products run whole and for the k ranges of split-k, and the
// rule that picks one.  Every tile sums k in the same order, so the pick changes
// the time of a product and never its bits.
#include <algorithm>

#include "pipe_gemm.h"

namespace mgemm {

// Tile blockIdx.x of C over the k range blockIdx.y (kc values, a multiple of every
// BK; kc = k for a product run whole).  W == NULL: into C with alpha and beta;
// else the partial product, alpha = 1 and beta = 0, into plane blockIdx.y of W (m x
// n, row stride n).
//
// Bound: the matrix cores, and between k-steps the barrier and the first LDS reads.
// Two stages of 18-36 KB leave room for two to eight work-groups per compute unit,
// whose products fill each other's barriers, prologues and epilogues: with FP64
// 1999 x 1501 x 2777 (odd rows) the two-stage register-staged 64 x 64 x 32 tile ran
// at 37.6 TFLOP/s, this 64 x 64 x 16 tile at 62.
template <typename T, int BM, int BN, int BK, int OCC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC)))
gemm_direct_kernel(GemmArgs p, int64_t kc, T *W) {
    typedef PipeShape<T, BM, BN, BK, 2, 2> S;
    __shared__ u32x4_t lds[2 * S::STAGE];
    const int tiles_m = (int)((p.m + BM - 1) / BM);
    const int tiles_n = (int)((p.n + BN - 1) / BN);
    int tm, tn;
    tile_of_block(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    if (W) {
        const int64_t y = blockIdx.y, k0 = y * kc;
        p.A = (const T *)p.A + k0;
        p.B = (const T *)p.B + k0 * p.ldb;
        p.C = W + y * p.m * p.n;
        p.ldc = p.n;
        p.k = p.k - k0 < kc ? p.k - k0 : kc;
        p.alpha = 1.0;
        p.beta = 0.0;
    }
    pipe_tile<T, BM, BN, BK, 2, 2, 2>(p, lds, (int64_t)tm * BM, (int64_t)tn * BN);
}

template <typename T, int BM, int BN, int BK, int OCC>
static hipError_t launch_direct(const GemmArgs &a, int S, int64_t kc, void *W, hipStream_t s) {
    const int64_t blocks = ((a.m + BM - 1) / BM) * ((a.n + BN - 1) / BN);
    if (blocks <= 0) return hipSuccess;
    if (!grid_fits(blocks, DIRECT_THREADS) || S < 1 || S > 65535) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_direct_kernel<T, BM, BN, BK, OCC>), dim3((unsigned)blocks, (unsigned)S),
                       dim3(256), 0, s, a, kc, (T *)W);
    return hipGetLastError();
}

// Several whole products in one launch, described in the kernel's arguments (no copy
// to the device, nothing kept between calls): work-group b runs a tile of the problem
// whose tiles start at or before b.
struct ListProblem {
    const void *A, *B;
    void *C;
    double alpha, beta;
    int32_t m, n, k, lda, ldb, ldc;
};

struct ListArgs {
    int32_t count;
    int32_t first[LIST_MAX];                  // first tile of each problem
    ListProblem p[LIST_MAX];
};

template <typename T, int BM, int BN, int BK, int OCC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC)))
gemm_list_kernel(ListArgs a) {
    typedef PipeShape<T, BM, BN, BK, 2, 2> S;
    static_assert(LIST_MAX <= 64, "one lane per problem");
    __shared__ u32x4_t lds[2 * S::STAGE];
    const int lane = threadIdx.x & 63, bid = (int)blockIdx.x;
    const bool at = lane < a.count && a.first[lane < LIST_MAX ? lane : 0] <= bid;
    const int pi = __builtin_amdgcn_readfirstlane(__popcll(__ballot(at)) - 1);
    const ListProblem &q = a.p[pi];
    const int tiles_n = (q.n + BN - 1) / BN, local = bid - a.first[pi];
    const int tm = local / tiles_n, tn = local - tm * tiles_n;
    const GemmArgs g{q.m, q.n, q.k, q.alpha, q.beta, q.A, q.lda, q.B, q.ldb, q.C, q.ldc};
    pipe_tile<T, BM, BN, BK, 2, 2, 2>(g, lds, (int64_t)tm * BM, (int64_t)tn * BN);
}

template <typename T, int BM, int BN, int BK, int OCC>
static hipError_t launch_list(const GemmArgs *p, int count, hipStream_t s) {
    ListArgs a;
    a.count = count;
    int64_t tiles = 0;
    for (int i = 0; i < count; ++i) {
        const GemmArgs &g = p[i];
        a.first[i] = (int32_t)tiles;
        a.p[i] = {g.A, g.B, g.C, g.alpha, g.beta, (int32_t)g.m, (int32_t)g.n, (int32_t)g.k,
                  (int32_t)g.lda, (int32_t)g.ldb, (int32_t)g.ldc};
        tiles += ((g.m + BM - 1) / BM) * ((g.n + BN - 1) / BN);
    }
    if (!grid_fits(tiles, DIRECT_THREADS)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_list_kernel<T, BM, BN, BK, OCC>), dim3((unsigned)tiles), dim3(256), 0,
                       s, a);
    return hipGetLastError();
}

// The tiles of direct_tiles() (host_rules.h) and their launchers, in the same order.
struct DirectTile {
    TileCost c;
    hipError_t (*launch)(const GemmArgs &, int, int64_t, void *, hipStream_t);
    bool (*eligible)(const GemmArgs &);
    hipError_t (*list)(const GemmArgs *, int, hipStream_t);
};

#define DIRECT(COSTS, I, T, OCC) \
    {COSTS[I], &launch_direct<T, COSTS[I].bm, COSTS[I].bn, COSTS[I].bk, OCC>, \
     &pipe_eligible<T, COSTS[I].bm, COSTS[I].bn, COSTS[I].bk>, \
     &launch_list<T, COSTS[I].bm, COSTS[I].bn, COSTS[I].bk, OCC>}

static const DirectTile kDirectF64[DIRECT_TILES] = {
    DIRECT(kTileCostsF64, 0, double, 2), DIRECT(kTileCostsF64, 1, double, 2),
    DIRECT(kTileCostsF64, 2, double, 4), DIRECT(kTileCostsF64, 3, double, 4),
    DIRECT(kTileCostsF64, 4, double, 4), DIRECT(kTileCostsF64, 5, double, 4),
};

static const DirectTile kDirectF32[DIRECT_TILES] = {
    DIRECT(kTileCostsF32, 0, float, 2), DIRECT(kTileCostsF32, 1, float, 2),
    DIRECT(kTileCostsF32, 2, float, 3), DIRECT(kTileCostsF32, 3, float, 4),
    DIRECT(kTileCostsF32, 4, float, 4), DIRECT(kTileCostsF32, 5, float, 4),
};

hipError_t run_direct(const GemmArgs &a, int32_t dtype, int S, int64_t kc, void *W, int cus,
                      hipStream_t s, bool *ran) {
    const DirectTile *t = dtype == MGEMM_F32 ? kDirectF32 : kDirectF64;
    const DirectTile *best = nullptr;
    double tb = 0.0;
    if (cus <= 0) cus = 256;
    for (int i = 0; i < DIRECT_TILES; ++i) {
        if (!t[i].eligible(a) || !grid_fits(tiles_of(t[i].c, a.m, a.n), DIRECT_THREADS) ||
            !tile_taken(t[i].c, a.m, a.n, a.k, S, cus))
            continue;
        const double ti = tile_time(t[i].c, a.m, a.n, a.k, S, kc, cus);
        if (!best || ti < tb) {
            best = &t[i];
            tb = ti;
        }
    }
    *ran = best != nullptr;
    return best ? best->launch(a, S, kc, W, s) : hipSuccess;
}

bool list_eligible(const GemmArgs &a, int32_t dtype) {
    return list_joins((int64_t)elem_size(dtype), a.m, a.n, a.k, a.A, a.lda, a.B, a.ldb, a.ldc);
}

// The products (list_eligible, any order) in launches of up to LIST_MAX, longest k
// first, each launch on the tile with the least estimate: its tiles' shares of the
// busy compute units, but no less than its longest tile alone.
hipError_t run_direct_list(const GemmArgs *p, int64_t count, int32_t dtype, int cus, hipStream_t s) {
    const DirectTile *t = dtype == MGEMM_F32 ? kDirectF32 : kDirectF64;
    if (cus <= 0) cus = 256;
    for (int64_t i0 = 0; i0 < count; i0 += LIST_MAX) {
        const int c = (int)std::min<int64_t>(LIST_MAX, count - i0);
        const DirectTile *best = nullptr;
        double tb = 0.0;
        for (int i = 0; i < DIRECT_TILES; ++i) {
            const TileCost &d = t[i].c;
            const double area = d.bm * d.bn / 4096.0;
            double sum = 0.0, longest = 0.0;
            for (int j = 0; j < c; ++j) {
                const GemmArgs &g = p[i0 + j];
                const double tiles = (double)((g.m + d.bm - 1) / d.bm) * (double)((g.n + d.bn - 1) / d.bn);
                const double ks = (double)((g.k + d.bk - 1) / d.bk * d.bk);
                sum += tiles * (d.each + d.rate * ks * area * (d.alone / d.resident + 1.0));
                longest = std::max(longest, d.each + d.rate * ks * area * (d.alone + 1.0));
            }
            const double ti = d.start + std::max(sum / cus, longest);
            if (!best || ti < tb) {
                best = &t[i];
                tb = ti;
            }
        }
        const hipError_t he = best->list(p + i0, c, s);
        if (he != hipSuccess) return he;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Many products in one launch (the default batched plan).
// ---------------------------------------------------------------------------
// Work-group b runs entry b / BATCH_LISTS of list b % BATCH_LISTS of the tile map (the
// hardware deals consecutive work-groups to the XCDs in turn, so a list's tiles share
// the panels of A and B in one L2); the hardware replaces a finished work-group by the
// next one, so short tiles need no queue of their own.
//
// Bound: the matrix cores for the large products, the load latency of a tile's first
// k-steps for the small ones, which four work-groups per compute unit hide.
template <typename T, int BM, int BN, int BK, int OCC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC)))
gemm_batched_direct_kernel(const BatchProblem *__restrict__ probs,
                           const uint64_t *__restrict__ map, const int64_t *__restrict__ off) {
    typedef PipeShape<T, BM, BN, BK, 2, 2> S;
    __shared__ u32x4_t lds[2 * S::STAGE];
    const unsigned list = blockIdx.x % BATCH_LISTS;
    const int64_t idx = off[list] + (int64_t)(blockIdx.x / BATCH_LISTS);
    if (idx >= off[list + 1]) return;
    const uint64_t e = map[idx];
    constexpr uint64_t RC = (1ull << TILE_MAP_RC_BITS) - 1;
    const int64_t tm = (int64_t)((e >> TILE_MAP_RC_BITS) & RC), tn = (int64_t)(e & RC);
    const GemmArgs g = probs[e >> (2 * TILE_MAP_RC_BITS)].g;
    pipe_tile<T, BM, BN, BK, 2, 2, 2>(g, lds, tm * BM, tn * BN);
}

bool batched_direct_eligible(const GemmArgs &a, int32_t dtype) {
    return dtype == MGEMM_F32 ? pipe_eligible<float, 64, 64, 32>(a)
                              : pipe_eligible<double, 64, 64, 16>(a);
}

hipError_t launch_batched_direct(int32_t dtype, const BatchProblem *probs, const uint64_t *map,
                                 const int64_t *off, int64_t longest, hipStream_t s) {
    const int64_t blocks = longest * BATCH_LISTS;
    if (blocks <= 0) return hipSuccess;
    if (!grid_fits(blocks, DIRECT_THREADS)) return hipErrorInvalidConfiguration;
    if (dtype == MGEMM_F32)
        hipLaunchKernelGGL((gemm_batched_direct_kernel<float, 64, 64, 32, 3>),
                           dim3((unsigned)blocks), dim3(256), 0, s, probs, map, off);
    else
        hipLaunchKernelGGL((gemm_batched_direct_kernel<double, 64, 64, 16, 4>),
                           dim3((unsigned)blocks), dim3(256), 0, s, probs, map, off);
    return hipGetLastError();
}

}  // namespace mgemm
