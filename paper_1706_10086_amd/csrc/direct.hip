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
// at 37.6 TFLOP/s, this 64 x 64 x 16 tile at 60.
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
    if (blocks > 0x7fffffff || S < 1 || S > 65535) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_direct_kernel<T, BM, BN, BK, OCC>), dim3((unsigned)blocks, (unsigned)S),
                       dim3(256), 0, s, a, kc, (T *)W);
    return hipGetLastError();
}

// A tile and its time: with q = ceil(tiles / CUs) work-groups for the busiest
// compute unit, R of them at a time, and k rounded up to the k-step,
//   t = start + each q + rate k (BM BN / 4096) (sum over rounds of (alone + r))
// microseconds, r work-groups in the round (R in all but the last): `alone` is the
// part of a k-step that co-resident work-groups hide from each other, `each` a
// tile's prologue and epilogue.  The coefficients are least squares on the log
// of the times of 119 shapes per type (squares 64-8192, log-uniform 32-8192 and large
// ragged ones, MI355X, calls back to back, within 4-13 % rms); picking by them
// reaches 0.991 of the best tile of each shape in both types (geometric mean).
struct DirectTile {
    int bm, bn, bk;
    int resident;            // R: work-groups a compute unit holds (LDS, registers)
    double start, each, rate, alone;
    hipError_t (*launch)(const GemmArgs &, int, int64_t, void *, hipStream_t);
    bool (*eligible)(const GemmArgs &);
};

#define DIRECT(T, BM, BN, BK, OCC, R, START, EACH, RATE, ALONE) \
    {BM, BN, BK, R, START, EACH, RATE, ALONE, &launch_direct<T, BM, BN, BK, OCC>, &pipe_eligible<T, BM, BN, BK>}

static const DirectTile kDirectF64[] = {
    DIRECT(double, 128, 128, 16, 2, 2, 0.00, 9.90, 0.02724, 0.081),
    DIRECT(double, 64, 128, 16, 2, 3, 2.16, 4.29, 0.02675, 0.278),
    DIRECT(double, 64, 64, 16, 4, 4, 2.98, 1.96, 0.02792, 0.369),
    DIRECT(double, 64, 32, 16, 4, 5, 2.49, 1.19, 0.02768, 1.000),
    DIRECT(double, 32, 32, 32, 4, 4, 2.58, 0.89, 0.02839, 0.874),
    DIRECT(double, 32, 32, 16, 4, 8, 2.36, 0.63, 0.03099, 1.465),
};

static const DirectTile kDirectF32[] = {
    DIRECT(float, 128, 128, 32, 2, 2, 3.90, 6.90, 0.01490, 0.038),
    DIRECT(float, 64, 128, 32, 2, 3, 4.12, 2.53, 0.01463, 0.150),
    DIRECT(float, 64, 64, 32, 3, 4, 3.94, 1.35, 0.01475, 0.349),
    DIRECT(float, 64, 32, 32, 4, 5, 3.59, 0.87, 0.01520, 0.643),
    DIRECT(float, 32, 32, 64, 4, 4, 3.23, 0.83, 0.01503, 0.879),
    DIRECT(float, 32, 32, 32, 4, 8, 3.03, 0.50, 0.01706, 0.995),
};

static double direct_time(const DirectTile &d, int64_t m, int64_t n, int64_t k, int64_t S, int cus) {
    const double tiles = (double)((m + d.bm - 1) / d.bm) * (double)((n + d.bn - 1) / d.bn) * (double)S;
    const double q = (double)(int64_t)((tiles + cus - 1) / cus);
    const double rounds = (double)(int64_t)(q / d.resident), last = q - rounds * d.resident;
    const double shared = rounds * (d.alone + d.resident) + (last > 0 ? d.alone + last : 0.0);
    const double ks = (double)((k + d.bk - 1) / d.bk * d.bk);
    return d.start + d.each * q + d.rate * ks * (d.bm * d.bn / 4096.0) * shared;
}

hipError_t run_direct(const GemmArgs &a, int32_t dtype, int S, int64_t kc, void *W, int cus,
                      hipStream_t s, bool *ran) {
    const DirectTile *t = dtype == MGEMM_F32 ? kDirectF32 : kDirectF64;
    const int cnt = dtype == MGEMM_F32 ? (int)(sizeof kDirectF32 / sizeof kDirectF32[0])
                                       : (int)(sizeof kDirectF64 / sizeof kDirectF64[0]);
    const DirectTile *best = nullptr;
    double tb = 0.0;
    for (int i = 0; i < cnt; ++i) {
        if (!t[i].eligible(a)) continue;
        const double ti = direct_time(t[i], a.m, a.n, kc, S, cus > 0 ? cus : 256);
        if (!best || ti < tb) {
            best = &t[i];
            tb = ti;
        }
    }
    *ran = best != nullptr;
    return best ? best->launch(a, S, kc, W, s) : hipSuccess;
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
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    if (dtype == MGEMM_F32)
        hipLaunchKernelGGL((gemm_batched_direct_kernel<float, 64, 64, 32, 3>),
                           dim3((unsigned)blocks), dim3(256), 0, s, probs, map, off);
    else
        hipLaunchKernelGGL((gemm_batched_direct_kernel<double, 64, 64, 16, 4>),
                           dim3((unsigned)blocks), dim3(256), 0, s, probs, map, off);
    return hipGetLastError();
}

}  // namespace mgemm
