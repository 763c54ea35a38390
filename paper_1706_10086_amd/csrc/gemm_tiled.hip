// Tiled GEMM C = alpha*A*B + beta*C on gfx950 matrix cores, FP64 and FP32.
//
// The computation is the paper's tiled GEMM (Sec. 2.1, Fig. 2): each work-group
// owns one tile of C (Sec. 2.1: one C tile per block, the grid of Eq. 3 becoming
// ceil(m/BM) x ceil(n/BN) work-groups); an outer loop walks the k-dimension in
// steps of BK, staging one BM x BK tile of A and one BK x BN tile of B in LDS (the
// tile cache of Eq. 5, here (BM*BK + BK*BN) * S bytes per stage); an inner loop
// multiplies the staged tiles into a per-thread register sub-tile of C (the
// thread-local temporary C tile of Fig. 2, the multiply-add of Listing 2); C is
// read and written once at the end (the streamed epilogue of Fig. 2).
//
// gfx950 specifics (not from the paper):
//  * the inner multiply runs on MFMA: v_mfma_f64_16x16x4_f64 for FP64 and
//    v_mfma_f32_16x16x4_f32 for FP32, each wave owning a WM x WN block of C held
//    as (WM/16) x (WN/16) accumulator fragments;
//  * one lane of an MFMA fragment reads two consecutive k values of A with one
//    16-byte LDS read and feeds them to two MFMAs; B supplies the same two k rows,
//    so the k-sum is complete, only reordered;
//  * LDS rows are padded so the fragment reads are free of bank conflicts;
//  * global loads are coalesced runs of EPT consecutive elements per thread, and
//    with double buffering the next k-step's loads are in flight while the
//    current step is multiplied;
//  * work-group ids are remapped so that the work-groups placed on one XCD (the
//    hardware deals ids round-robin over the 8 XCDs) own a compact group of C
//    tiles and share their A and B panels in that XCD's L2.
#include <algorithm>
#include <vector>

#include "grid_registry.h"
#include "pipe_gemm.h"

namespace mgemm {

// Many GEMMs sharing one configuration: a persistent grid whose work-groups take
// work items from atomic counters until every list is exhausted.  With a tile
// map (item = map entry: problem, tile row, tile column) there is one list per
// XCD, each holding whole problems or runs of a problem's tiles, so the panels of
// A and B that a run of tiles shares stay in that XCD's L2; a work-group drains
// its own XCD's list, then takes from the others.  Without a map the single list
// holds tile numbers (problems numbered tile by tile, BatchProblem::tile0 the
// first of each) and a tile's problem is found by binary search.  Lists order
// their problems by decreasing work.  Thread 0 asks for the next item as the
// work-group starts a tile, so the atomic's latency hides behind the tile's work.
// Split-k partial products: work-group (x, y) computes C tile x over the y-th
// range of kc values of k (columns of A, rows of B) with alpha = 1 and beta = 0,
// into plane y of W (m x n, row stride n); splitk_reduce_kernel sums the planes.
// A range starts at a multiple of kc (a multiple of BK), so rows keep the
// alignment of A and B.
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int EPT, int DBUF, int OCC,
          bool ALIGN>
__global__ void __launch_bounds__(64 * WGM * WGN)
__attribute__((amdgpu_waves_per_eu(OCC > 0 ? OCC : 1)))
gemm_splitk_kernel(GemmArgs p, int64_t kc, T *W) {
    typedef TileLds<T, BM, BN, BK, DBUF> L;
    constexpr int PAD = occupancy_pad_elems<T>(OCC, WGM * WGN,
                                               (L::A_ELEMS + L::B_ELEMS) * (int)sizeof(T));
    __shared__ __attribute__((aligned(16))) T sA[L::A_ELEMS + PAD];
    __shared__ __attribute__((aligned(16))) T sB[L::B_ELEMS];
    const int tiles_m = (int)((p.m + BM - 1) / BM);
    const int tiles_n = (int)((p.n + BN - 1) / BN);
    int tm, tn;
    tile_of_block(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    const int64_t y = blockIdx.y, k0 = y * kc;
    GemmArgs q = p;
    q.k = p.k - k0 < kc ? p.k - k0 : kc;
    q.A = (const T *)p.A + k0;
    q.B = (const T *)p.B + k0 * p.ldb;
    q.alpha = 1.0;
    q.beta = 0.0;
    q.C = W + y * p.m * p.n;
    q.ldc = p.n;
    tile_gemm<T, BM, BN, BK, WGM, WGN, EPT, DBUF, ALIGN>(q, (int64_t)tm * BM, (int64_t)tn * BN,
                                                          sA, sB);
}

// C = alpha * (W_0 + W_1 + ... + W_{S-1}) + beta * C, the planes added in order
// (the same rounding of alpha and beta as the tile epilogue).  Columns run over
// blockIdx.x and a row of threads (coalesced), rows over blockIdx.y and the rows of
// threads: up to four rows of narrow results to a work-group.
//
// Bound: the latency of the planes' loads, so S is a template parameter and all of an
// element's loads are in flight at once, and for narrow results the work-groups'
// start.  FP32 10880 x 68, 3 planes: 5.7 us; one row to a work-group 10.1, with S a
// loop count 9.0, and loading seven planes at a time and the rest in turn 17.4.  FP64
// 300 x 129, 14 planes: 4.2 (5.5 with the loop).
template <typename T, int S>
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const T *__restrict__ W, int64_t m, int64_t n, T alpha, T beta, int read_c,
                     T *C, int64_t ldc) {
    const int64_t plane = m * n;
    for (int64_t row = (int64_t)blockIdx.y * blockDim.y + threadIdx.y; row < m;
         row += (int64_t)gridDim.y * blockDim.y)
        for (int64_t col = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; col < n;
             col += (int64_t)gridDim.x * blockDim.x) {
            const int64_t i = row * n + col;
            T *c = C + row * ldc + col;
            T w[S];
#pragma unroll
            for (int y = 0; y < S; ++y) w[y] = W[y * plane + i];
            const T cv = read_c ? *c : (T)0;
            T acc = w[0];
#pragma unroll
            for (int y = 1; y < S; ++y) acc += w[y];
            *c = read_c ? scale_add(alpha, acc, beta, cv) : alpha * acc;
        }
}

// Waves per SIMD the batched kernel is compiled for: the configuration's
// occupancy if it names one; for the four-wave 64 x 64 x 16 tile three (it
// still fits without spilling, and a batch of short tiles is bound by load
// latency, which more resident work-groups hide; FP64 spills at four, FP32 fits
// four but ran no faster).
constexpr int batched_waves(int bm, int bn, int bk, int waves, int occ) {
    return occ > 0 ? occ : (bm * bn <= 64 * 64 && bk <= 16 && waves == 4 ? 3 : 1);
}

template <typename T, int BM, int BN, int BK, int WGM, int WGN, int EPT, int DBUF, int OCC>
__global__ void __launch_bounds__(64 * WGM * WGN)
__attribute__((amdgpu_waves_per_eu(batched_waves(BM, BN, BK, WGM * WGN, OCC))))
gemm_batched_kernel(const BatchProblem *__restrict__ probs, const uint64_t *__restrict__ tile_map,
                    const int64_t *__restrict__ list_off, int nlist, int nprob,
                    unsigned long long *counters) {
    typedef TileLds<T, BM, BN, BK, DBUF> L;
    __shared__ __attribute__((aligned(16))) T sA[L::A_ELEMS];
    __shared__ __attribute__((aligned(16))) T sB[L::B_ELEMS];
    __shared__ int64_t next;
    // the item index is uniform: keep it (and all that follows from it) in
    // scalar registers
    auto uniform_next = [&]() {
        const uint64_t tv = (uint64_t)next;
        return (int64_t)(((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(tv >> 32)) << 32) |
                         (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)tv));
    };
    // thread 0's state: lists visited so far and the counter value last taken
    const int home = (int)(blockIdx.x % (unsigned)nlist);
    int visit = 0;
    unsigned long long taken = 0;
    // (thread 0) the item that `taken` names, moving on to the next list while
    // the current one is exhausted; -1 once every list is
    auto settle = [&]() -> int64_t {
        for (;;) {
            const int l = home + visit < nlist ? home + visit : home + visit - nlist;
            const int64_t idx = list_off[l] + (int64_t)taken;
            if (idx < list_off[l + 1]) return idx;
            if (++visit >= nlist) return -1;
            const int l2 = home + visit < nlist ? home + visit : home + visit - nlist;
            taken = atomicAdd(&counters[l2], 1ull);
        }
    };
    if (threadIdx.x == 0) {
        taken = atomicAdd(&counters[home], 1ull);
        next = settle();
    }
    __syncthreads();
    int64_t t = uniform_next();
    while (t >= 0) {
        if (threadIdx.x == 0) {
            const int l = home + visit < nlist ? home + visit : home + visit - nlist;
            taken = atomicAdd(&counters[l], 1ull);                // read after this tile
        }
        int pi;
        int64_t tm, tn;
        if (tile_map) {
            const uint64_t e = tile_map[t];
            const uint64_t eu = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(e >> 32)) << 32) |
                                (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)e);
            constexpr uint64_t RC = (1ull << TILE_MAP_RC_BITS) - 1;
            pi = (int)(eu >> (2 * TILE_MAP_RC_BITS));
            tm = (int64_t)((eu >> TILE_MAP_RC_BITS) & RC);
            tn = (int64_t)(eu & RC);
        } else {
            int lo = 0, hi = nprob - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (probs[mid].tile0 <= t) lo = mid;
                else hi = mid - 1;
            }
            pi = lo;
            tm = tn = -1;
        }
        // copy the (uniform) descriptor word by word into scalar registers
        BatchProblem bp;
        {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(probs + pi);
            uint32_t *dst = reinterpret_cast<uint32_t *>(&bp);
#pragma unroll
            for (int w = 0; w < (int)(sizeof(BatchProblem) / 4); ++w)
                dst[w] = __builtin_amdgcn_readfirstlane(src[w]);
        }
        if (tm < 0) {
            const int64_t local = t - bp.tile0;
            tm = local / bp.tiles_n;
            tn = local - tm * bp.tiles_n;
        }
        // the tile runs gemm_ex's code for its problem's row alignment
        if (bp.aligned)
            tile_gemm<T, BM, BN, BK, WGM, WGN, EPT, DBUF, true, true>(bp.g, tm * BM, tn * BN, sA, sB);
        else
            tile_gemm<T, BM, BN, BK, WGM, WGN, EPT, DBUF, false, true>(bp.g, tm * BM, tn * BN, sA,
                                                                        sB);
        __syncthreads();                  // every wave has read the current index
        if (threadIdx.x == 0) next = settle();
        __syncthreads();
        t = uniform_next();
    }
}

// ---------------------------------------------------------------------------
// The direct-load tile of the registered configurations (double_buffer = 2).
// ---------------------------------------------------------------------------
// Two stages: a third one, of the same kernel with the loads two k-steps ahead,
// gave no tile more speed and takes the LDS of a second work-group (FP64 64 x 64
// x 32 at N = 4096 52 against 66 TFLOP/s with one and two work-groups per compute
// unit, 256 x 128 x 16 66 against 70).
constexpr int PIPE_STAGES = 2;

template <typename T, int BM, int BN, int BK, int WGM, int WGN>
__global__ void __launch_bounds__(64 * WGM * WGN)
    __attribute__((amdgpu_waves_per_eu(WGM * WGN / 4))) gemm_pipe_kernel(GemmArgs p) {
    typedef PipeShape<T, BM, BN, BK, WGM, WGN> S;
    __shared__ u32x4_t lds[PIPE_STAGES * S::STAGE];
    const int tiles_m = (int)((p.m + BM - 1) / BM);
    const int tiles_n = (int)((p.n + BN - 1) / BN);
    int tm, tn;
    tile_of_block(blockIdx.x, gridDim.x, tiles_m, tiles_n, tm, tn);
    pipe_tile<T, BM, BN, BK, WGM, WGN, PIPE_STAGES>(p, lds, (int64_t)tm * BM, (int64_t)tn * BN);
}

// ---------------------------------------------------------------------------
// Launchers and registries.
// ---------------------------------------------------------------------------
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int EPT, int DBUF, int OCC,
          bool ALIGN>
hipError_t launch_splitk(const GemmArgs &a, int S, int64_t kc, void *W, hipStream_t s) {
    int64_t blocks = ((a.m + BM - 1) / BM) * ((a.n + BN - 1) / BN);
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffff || S < 1 || S > 65535) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_splitk_kernel<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, ALIGN>),
                       dim3((unsigned)blocks, (unsigned)S), dim3(64 * WGM * WGN), 0, s, a, kc,
                       (T *)W);
    return hipGetLastError();
}

// Whether the plan may cut k on 128 x 128 tiles: rows of whole 16-byte loads on
// 16-byte bases and 32-bit panel offsets.
bool pipe_splitk_eligible(const GemmArgs &a, int32_t dtype) {
    const int64_t es = dtype == MGEMM_F32 ? 4 : 8;
    const int64_t EPU = 16 / es, BM = 128, BN = 128, BK = dtype == MGEMM_F32 ? 32 : 16;
    return a.k >= 1 && a.n >= EPU && a.n % EPU == 0 && a.lda % EPU == 0 && a.ldb % EPU == 0 &&
           ((uintptr_t)a.A % 16) == 0 && ((uintptr_t)a.B % 16) == 0 &&
           BM * a.lda * es < ((int64_t)1 << 31) && (BK * a.ldb + BN) * es < ((int64_t)1 << 31);
}

constexpr int REDUCE_PLANES_MAX = 16;

template <typename T, int S = 2>
static hipError_t reduce_planes(const T *W, int planes, const GemmArgs &a, hipStream_t s) {
    if (planes == S) {
        const int64_t tx = std::min<int64_t>((a.n + 63) / 64 * 64, 256), ty = 256 / tx;
        const int64_t gx = std::min<int64_t>((a.n + tx - 1) / tx, 64);
        const int64_t gy = std::min<int64_t>((a.m + ty - 1) / ty, 65535);
        hipLaunchKernelGGL((splitk_reduce_kernel<T, S>), dim3((unsigned)gx, (unsigned)gy),
                           dim3((unsigned)tx, (unsigned)ty), 0, s, W, a.m, a.n, (T)a.alpha, (T)a.beta,
                           a.beta != 0.0, (T *)a.C, a.ldc);
        return hipGetLastError();
    }
    if constexpr (S < REDUCE_PLANES_MAX) return reduce_planes<T, S + 1>(W, planes, a, s);
    return hipErrorInvalidConfiguration;
}

hipError_t splitk_reduce(int32_t dtype, const void *W, int S, const GemmArgs &a, hipStream_t s) {
    return dtype == MGEMM_F32 ? reduce_planes((const float *)W, S, a, s)
                              : reduce_planes((const double *)W, S, a, s);
}

template <typename T, int BM, int BN, int BK, int WGM, int WGN, int EPT, int DBUF, int OCC>
hipError_t launch_batched(const BatchProblem *probs, const uint64_t *tile_map,
                          const int64_t *list_off, int nlist, int nprob,
                          unsigned long long *counters, int grid, hipStream_t s) {
    hipLaunchKernelGGL((gemm_batched_kernel<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC>),
                       dim3((unsigned)grid), dim3(64 * WGM * WGN), 0, s, probs, tile_map, list_off,
                       nlist, nprob, counters);
    return hipGetLastError();
}

// Resident work-groups per compute unit of the batched kernel (occupancy query).
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int EPT, int DBUF, int OCC>
int batched_occupancy() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, gemm_batched_kernel<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC>,
            64 * WGM * WGN, 0) != hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

// The direct-load kernel where its requirements hold (pipe_eligible), else the
// two-stage kernel of the same tile (FWGM x FWGN waves), which sums in the same
// order.
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int FWGM, int FWGN, int FEPT,
          bool ALIGN>
hipError_t launch_pipe(const GemmArgs &a, hipStream_t s) {
    if (!pipe_eligible<T, BM, BN, BK>(a))
        return launch_tiled<T, BM, BN, BK, FWGM, FWGN, FEPT, 1, 0, ALIGN>(a, s);
    int64_t blocks = ((a.m + BM - 1) / BM) * ((a.n + BN - 1) / BN);
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_pipe_kernel<T, BM, BN, BK, WGM, WGN>), dim3((unsigned)blocks),
                       dim3(64 * WGM * WGN), 0, s, a);
    return hipGetLastError();
}

// Registry entry of a direct-load configuration (double_buffer = 2); batched plans
// and large products from host memory use the two-stage kernel of the same tile.
// Its elems_per_thread is the elements of one 16-byte direct load; FWGM, FWGN and
// FEPT name the two-stage fallback (registered on its own as well).
#define MGEMM_PIPE_CFG(T, BM, BN, BK, WGM, WGN, FWGM, FWGN, FEPT)                      \
    {{BM, BN, BK, WGM * WGN, 16 / (int)sizeof(T), 2, WGM * WGN / 4},                      \
     &launch_pipe<T, BM, BN, BK, WGM, WGN, FWGM, FWGN, FEPT, true>,                       \
     &launch_pipe<T, BM, BN, BK, WGM, WGN, FWGM, FWGN, FEPT, false>,                      \
     &launch_batched<T, BM, BN, BK, FWGM, FWGN, FEPT, 1, 0>,                               \
     &batched_occupancy<T, BM, BN, BK, FWGM, FWGN, FEPT, 1, 0>,                            \
     {nullptr, nullptr},                                                                  \
     {&launch_tiled<T, BM, BN, BK, FWGM, FWGN, FEPT, 1, 0, true>,                         \
      &launch_tiled<T, BM, BN, BK, FWGM, FWGN, FEPT, 1, 0, false>}}

// A two-stage configuration that also runs split-k for the built-in choice (FP64
// only: at N = 1024 it raised FP64 from 27.0 to 30.9 TFLOP/s, while FP32, twice as
// fast per tile, lost 4 % to the extra reduction).
#define MGEMM_REG_SPLITK(T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC)                       \
    {{BM, BN, BK, WGM * WGN, EPT, DBUF, OCC},                                             \
     &launch_tiled<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, true>,                        \
     &launch_tiled<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, false>,                       \
     &launch_batched<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC>,                             \
     &batched_occupancy<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC>,                          \
     {&launch_splitk<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, true>,                      \
      &launch_splitk<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, false>}}

#define MGEMM_CFG(T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC)                              \
    {{BM, BN, BK, WGM * WGN, EPT, DBUF, OCC},                                             \
     &launch_tiled<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, true>,                        \
     &launch_tiled<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC, false>,                       \
     &launch_batched<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC>,                             \
     &batched_occupancy<T, BM, BN, BK, WGM, WGN, EPT, DBUF, OCC>}

// (the 128 x 128 x 16 tile compiled for two waves per SIMD, one or two stages,
// spilled registers to scratch and is not registered)
static const KernelEntry kF64[] = {
    MGEMM_CFG(double, 128, 128, 16, 2, 2, 2, 1, 0),
    MGEMM_CFG(double, 128, 128, 32, 2, 2, 4, 1, 0),
    MGEMM_CFG(double, 256, 128, 16, 4, 2, 2, 1, 0),
    MGEMM_CFG(double, 128, 256, 16, 2, 4, 2, 1, 0),
    MGEMM_CFG(double, 128, 64, 16, 2, 2, 2, 1, 0),
    MGEMM_CFG(double, 128, 64, 32, 2, 2, 4, 0, 2),
    MGEMM_REG_SPLITK(double, 64, 64, 16, 2, 2, 2, 1, 0),
    MGEMM_CFG(double, 64, 64, 32, 2, 2, 2, 1, 0),
    MGEMM_REG_SPLITK(double, 32, 32, 16, 1, 1, 2, 1, 0),
    // direct-load kernels: the two large tiles with two waves per SIMD,
    // and a 64 x 64 tile with one (for products of a few hundred tiles: at 1024^3 it
    // ran at 47 TFLOP/s against 37 for the best two-stage tile; 64 x 64 x 16 reached
    // 40, 128 x 128 with four waves and 128 x 64 tiles 17-29)
    MGEMM_PIPE_CFG(double, 256, 128, 16, 4, 2, 4, 2, 2),
    MGEMM_PIPE_CFG(double, 128, 128, 16, 4, 2, 2, 2, 2),
    MGEMM_PIPE_CFG(double, 64, 64, 32, 2, 2, 2, 2, 4),
};

static const KernelEntry kF32[] = {
    MGEMM_CFG(float, 128, 128, 16, 2, 2, 2, 1, 0),
    MGEMM_CFG(float, 128, 128, 32, 2, 2, 4, 1, 0),
    MGEMM_CFG(float, 128, 128, 32, 2, 2, 4, 1, 2),
    MGEMM_CFG(float, 256, 128, 32, 4, 2, 4, 1, 0),
    MGEMM_CFG(float, 128, 256, 32, 2, 4, 4, 1, 0),
    MGEMM_CFG(float, 128, 64, 32, 2, 2, 4, 1, 0),
    MGEMM_CFG(float, 64, 64, 16, 2, 2, 2, 1, 0),
    MGEMM_CFG(float, 32, 32, 16, 1, 1, 2, 1, 0),
    MGEMM_PIPE_CFG(float, 256, 128, 32, 4, 2, 4, 2, 4),
    MGEMM_PIPE_CFG(float, 128, 128, 32, 4, 2, 2, 2, 4),
    // one wave per SIMD, 64 x 64 (1024^3: 89 TFLOP/s with k-steps of 64, 82 with 32,
    // against 62 for the best two-stage tile)
    MGEMM_PIPE_CFG(float, 64, 64, 64, 2, 2, 2, 2, 4),
    MGEMM_PIPE_CFG(float, 64, 64, 32, 2, 2, 2, 2, 4),
};

// The hand-registered entries followed by every part of the tuning grid.
static std::vector<KernelEntry> joined(const KernelEntry *hand, size_t nh,
                                       const GridPartFn *parts) {
    std::vector<KernelEntry> all(hand, hand + nh);
    for (int p = 0; p < GRID_PARTS; ++p) {
        int cnt = 0;
        const KernelEntry *e = parts[p](&cnt);
        all.insert(all.end(), e, e + cnt);
    }
    return all;
}

const KernelEntry *f64_registry(int *count) {
    static const std::vector<KernelEntry> all =
        joined(kF64, sizeof(kF64) / sizeof(kF64[0]), kGridF64Parts);
    *count = (int)all.size();
    return all.data();
}

const KernelEntry *f32_registry(int *count) {
    static const std::vector<KernelEntry> all =
        joined(kF32, sizeof(kF32) / sizeof(kF32[0]), kGridF32Parts);
    *count = (int)all.size();
    return all.data();
}

}  // namespace mgemm
