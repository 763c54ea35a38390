// The direct-load tiled GEMM of one C tile (pipe_tile): k-steps are copied
// straight from global memory into LDS stages, for rows of any alignment.  Shared
// by the single-GEMM, split-k and batched kernels.
#pragma once

#include <type_traits>

#include "tile_gemm.h"

namespace mgemm {

// ---------------------------------------------------------------------------
// Shape of one k-step in LDS.
// ---------------------------------------------------------------------------
// WGM x WGN waves, each owning a WM x WN block of C as (WM/16) x (WN/16)
// accumulator fragments; a stage holds BM padded rows of A, then BK padded rows of
// B, in 16-byte units.
template <typename T, int BM, int BN, int BK, int WGM, int WGN>
struct PipeShape {
    static constexpr int NT = 64 * WGM * WGN;
    static constexpr int WM = BM / WGM, WN = BN / WGN;
    static constexpr int FM = WM / 16, FN = WN / 16;
    static constexpr int G = BK / 8;                               // 8-deep k groups
    static constexpr int EPU = 16 / (int)sizeof(T);                // elements per unit
    static constexpr int ROW_A = BK * (int)sizeof(T) / 16;         // 16-byte units per A row
    static constexpr int AU = ROW_A + 1;                           // padded A row (units)
    static constexpr int ROW_B = BN * (int)sizeof(T) / 16;         // units per B row
    // padded B row: stride BN + 8 (FP64) elements, so the two k rows (2 kq apart)
    // one fragment read touches fall in distinct banks
    static constexpr int BU = ROW_B + (sizeof(T) == 8 ? 4 : 2);
    // the A region ends on a wave's load (64 units), so each load instruction of a
    // wave reads one operand and its panel address is wave-uniform
    static constexpr int A_UNITS = (BM * AU + 63) / 64 * 64;
    static constexpr int STAGE = A_UNITS + BK * BU;                // units per stage
    static constexpr int LOADS = (STAGE + NT - 1) / NT;            // load instructions per wave
};

// Whether pipe_tile can run a product with tiles of BM x BN x BK.
template <typename T, int BM, int BN, int BK>
inline bool pipe_eligible(const GemmArgs &a) {
    return direct_loads(sizeof(T), BM, BN, BK, a.m, a.n, a.k, a.A, a.lda, a.B, a.ldb);
}

// One BM x BN tile of C: rows from m0, columns [c0, c0 + BN) of which this tile
// stores those below n.  lds holds NST stages of PipeShape::STAGE units.
//
// Each k-step's A and B tiles are copied into a stage by global_load_lds (16 bytes
// per lane, no staging registers).  While the products of k-step c run from
// registers, every fragment register is refilled with k-step c+1 right after its
// last use, and k-step c+NST loads into the stage whose contents all waves already
// hold in registers, so NST stages keep NST-1 k-steps in flight beside the one
// being read.  One barrier per k-step.  The k-sum order per element is
// gemm_tiled_kernel's, so both give bit-identical results (but for the sign of a sum
// that underflows to zero: the zeros that pad k to a whole k-step make it positive).
//
// Rows and columns need no alignment beyond 4 bytes (16-byte loads at 4-byte
// aligned addresses ran at the rate of aligned ones: 56-59 bytes per cycle and
// compute unit either way).  An overhanging column tile starts up to three columns
// earlier, so that its last 16-byte unit ends with the row (the columns before c0
// repeat the neighbour's and are not stored); rows >= m and units past n load
// clamped addresses whose products are not stored, and a wave whose whole part lies
// outside C runs no products.  A partial last k-step is loaded element-wise and
// zero-padded.  Where n < BN and n is no
// multiple of the unit (the first column tile cannot start earlier), the unit at the
// row's end also reads the first elements of the next row, so the last row of B stays
// with the element-wise step.
//
// The function ends with a barrier-free epilogue: a caller that reuses lds puts a
// barrier before the next tile.
template <typename T, int BM, int BN, int BK, int WGM, int WGN, int NST>
__device__ __forceinline__ void pipe_tile(const GemmArgs &p, u32x4_t *lds, int64_t m0, int64_t c0) {
    typedef PipeShape<T, BM, BN, BK, WGM, WGN> S;
    typedef Elem<T> E;
    typedef typename E::vec2 vec2;
    typedef typename E::acc4 acc4;
    static_assert(S::WM % 16 == 0 && S::WN % 16 == 0 && BK % 8 == 0, "tile shape");
    static_assert(NST >= 2, "one stage is read while another fills");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const AS_GLOBAL T *__restrict__ A = (const AS_GLOBAL T *)p.A;
    const AS_GLOBAL T *__restrict__ B = (const AS_GLOBAL T *)p.B;
    const int64_t lda = p.lda, ldb = p.ldb;
    // columns: the tile covers [n0, n0 + BN) and stores those from c0 on; an
    // overhanging tile starts up to a unit earlier, so that units end with the row
    const int first_col =
        c0 > 0 && p.n - c0 < BN ? (int)((S::EPU - (p.n - c0) % S::EPU) % S::EPU) : 0;
    const int64_t n0 = c0 - first_col;
    const int64_t mrem = p.m - m0, nrem = p.n - n0;
    // whether any row and column of this wave's part lie inside C (uniform)
    const bool live = mrem > wm * S::WM && nrem > wn * S::WN;

    // Per-lane source byte offsets of each load instruction, relative to the
    // tile's A panel (A + m0*lda) or B panel (B + n0) at k-step 0 (32 bits:
    // pipe_eligible).
    const int mlast = mrem < BM ? (int)mrem - 1 : BM - 1;
    const int nlast = nrem < BN ? (int)nrem : BN;
    const uint32_t lda_b = (uint32_t)(lda * (int64_t)sizeof(T));
    const uint32_t ldb_b = (uint32_t)(ldb * (int64_t)sizeof(T));
    uint32_t src_off[S::LOADS];
#pragma unroll
    for (int i = 0; i < S::LOADS; ++i) {
        const int u = i * S::NT + tid;
        if (u < S::A_UNITS) {
            const int r = u / S::AU, c = u % S::AU;
            src_off[i] = (uint32_t)(r < mlast ? r : mlast) * lda_b +
                         (uint32_t)(c < S::ROW_A ? c : S::ROW_A - 1) * 16u;
        } else {
            const int v = u - S::A_UNITS;
            const int r = v / S::BU, c = v % S::BU;
            int col = (c < S::ROW_B ? c : S::ROW_B - 1) * S::EPU;
            // a unit wholly past n reads the row's last whole unit instead
            if (col >= nlast) col = nlast - S::EPU;
            src_off[i] = (uint32_t)(r < BK ? r : BK - 1) * ldb_b + (uint32_t)col * (uint32_t)sizeof(T);
        }
    }
    const AS_GLOBAL char *Apanel = (const AS_GLOBAL char *)(A + m0 * lda);
    const AS_GLOBAL char *Bpanel = (const AS_GLOBAL char *)(B + n0);
    // load instruction i of k-step kstep into stage
    auto issue_one = [&](int i, int64_t kstep, u32x4_t *stage) {
        const int first = i * S::NT + wave * 64;
        // only the last instruction can run past the stage (uniform per wave)
        if ((i + 1) * S::NT > S::STAGE && first >= S::STAGE) return;
        // which operand: known at compile time but for the one instruction where
        // some waves load A and others B
        const bool in_a = (i + 1) * S::NT <= S::A_UNITS ||
                          (i * S::NT < S::A_UNITS && first < S::A_UNITS);
        const AS_GLOBAL char *src = in_a ? Apanel + kstep * (BK * (int64_t)sizeof(T))
                                         : Bpanel + kstep * (BK * ldb * (int64_t)sizeof(T));
        __builtin_amdgcn_global_load_lds((const AS_GLOBAL void *)(src + src_off[i]),
                                         (__attribute__((address_space(3))) void *)(stage + first),
                                         16, 0, 0);
    };
    auto issue = [&](int64_t kstep, u32x4_t *stage) {
#pragma unroll
        for (int i = 0; i < S::LOADS; ++i) issue_one(i, kstep, stage);
    };
    // waits until at most `steps` k-steps of this wave's loads are in flight
    const bool full_loads = S::STAGE % S::NT == 0 || (S::LOADS - 1) * S::NT + wave * 64 < S::STAGE;
    auto wait_steps = [&](auto steps) {
        constexpr int N = decltype(steps)::value;
        if (N == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        else if (full_loads) __builtin_amdgcn_s_waitcnt(vmcnt_imm(N * S::LOADS));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(N * (S::LOADS - 1)));
    };

    acc4 acc[S::FM][S::FN];
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j) acc[i][j] = acc4{0, 0, 0, 0};

    const int l16 = lane & 15, kq = lane >> 4;
    // A fragment (g, i): elements g*8 + 2kq, +1 of row wm*WM + i*16 + l16; B fragment
    // (g, h, j): element (g*8 + 2kq + h, wn*WN + j*16 + l16) of the B region
    const int a_elem = (wm * S::WM + l16) * S::AU * S::EPU + 2 * kq;
    const int b_elem = S::A_UNITS * S::EPU + (2 * kq) * S::BU * S::EPU + wn * S::WN + l16;
    vec2 af[S::G][S::FM];
    T bf[S::G][2][S::FN];
    auto read_a = [&](const u32x4_t *st, int g, int i) {
        af[g][i] = *(const vec2 *)((const T *)st + a_elem + i * 16 * S::AU * S::EPU + g * 8);
    };
    auto read_b = [&](const u32x4_t *st, int g, int h) {
        const T *stT = (const T *)st;
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
            bf[g][h][j] = stT[b_elem + (g * 8 + h) * S::BU * S::EPU + j * 16];
    };
    // products of one k-step; with REFILL each fragment is refilled from the next
    // stage right after its last use.  With LOAD the loads of k-step lk into stage
    // lst are spread over the products, one every few fragment rows, so the memory
    // pipeline takes a few at a time instead of every wave queueing all of them at
    // the barrier.
    auto products = [&](auto load, auto refill, const u32x4_t *nst, int64_t lk, u32x4_t *lst) {
        constexpr bool LOAD = decltype(load)::value, REFILL = decltype(refill)::value;
        constexpr int SLOTS = S::G * 2 * S::FM;
        constexpr int EVERY = SLOTS / S::LOADS > 0 ? SLOTS / S::LOADS : 1;
        constexpr int PER = (S::LOADS + SLOTS - 1) / SLOTS;        // loads per slot
        static_assert((S::LOADS - 1) / PER * EVERY < SLOTS, "every load gets a slot");
#pragma unroll
        for (int g = 0; g < S::G; ++g) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < S::FM; ++i) {
#pragma unroll
                    for (int j = 0; j < S::FN; ++j)
                        acc[i][j] = E::mma(af[g][i][h], bf[g][h][j], acc[i][j]);
                    if (REFILL && h == 1) read_a(nst, g, i);
                    const int slot = (g * 2 + h) * S::FM + i;
                    if (LOAD && slot % EVERY == 0) {
#pragma unroll
                        for (int q = 0; q < PER; ++q)
                            if (slot / EVERY * PER + q < S::LOADS)
                                issue_one(slot / EVERY * PER + q, lk, lst);
                    }
                    if (h == 1 || slot % EVERY == 0) __builtin_amdgcn_sched_barrier(0);
                }
                if (REFILL) read_b(nst, g, h);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // k-steps: nk full ones by direct loads; the rest (a partial last k-step, or a
    // whole one whose last row of B the direct loads must not take) element by
    // element, zero outside A and B (as the two-stage kernel pads)
    const bool row_end = nrem < BN && nrem % S::EPU != 0;
    const int64_t nk = row_end ? (p.k - 1) / BK : p.k / BK;
    const int ktail = (int)(p.k - nk * BK);
    constexpr int NA = BM * BK / S::NT, NB = BK * BN / S::NT;
    static_assert(NA * S::NT == BM * BK && NB * S::NT == BK * BN, "tail split");
    // Where 16 registers hold a thread's share of that step, it is loaded before the
    // loop, its latency hidden behind the full k-steps, and takes its stage within
    // the loop; for the larger tiles (which have no registers to spare: FP64 128 x 128
    // x 16 spilled) it follows the loop.
    constexpr bool EARLY_TAIL = (NA + NB) * (int)sizeof(T) <= 64;
    // With k-steps of 32 and more, a product of less than one runs only the groups of 8
    // that hold values (FP32 2047 x 12135 x 13: 41.5 us with all four groups and loads of
    // clamped elements in place of the rows of B past k, 36.0 so; FP64's two groups of
    // 64 x 64 x 16 have no registers left for the branch).
    constexpr bool GROUPS = S::G > 2;
    const int64_t steps = nk + (EARLY_TAIL && ktail && !(GROUPS && nk == 0) ? 1 : 0);
    T ta[NA], tb[NB];
    auto load_tail = [&]() {
        const AS_GLOBAL T *At = (const AS_GLOBAL T *)(Apanel + nk * (BK * (int64_t)sizeof(T)));
        const AS_GLOBAL T *Bt = (const AS_GLOBAL T *)(Bpanel + nk * (BK * ldb * (int64_t)sizeof(T)));
#pragma unroll
        for (int e = 0; e < NA; ++e) {
            const int r = (tid + e * S::NT) / BK, c = (tid + e * S::NT) % BK;
            ta[e] = (T)0;
            if (r <= mlast && c < ktail) ta[e] = At[(int64_t)r * lda + c];
        }
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int r = (tid + e * S::NT) / BN, c = (tid + e * S::NT) % BN;
            tb[e] = (T)0;
            if (r < ktail && c < nlast) tb[e] = Bt[(int64_t)r * ldb + c];
        }
    };
    auto store_tail = [&](u32x4_t *stage) {
        T *sT = (T *)stage;
#pragma unroll
        for (int e = 0; e < NA; ++e)
            sT[(tid + e * S::NT) / BK * S::AU * S::EPU + (tid + e * S::NT) % BK] = ta[e];
#pragma unroll
        for (int e = 0; e < NB; ++e)
            sT[S::A_UNITS * S::EPU + (tid + e * S::NT) / BN * S::BU * S::EPU +
               (tid + e * S::NT) % BN] = tb[e];
    };

    // k-step c sits in stage c % NST; the first NST are filled here
#pragma unroll
    for (int c = 0; c < NST; ++c)
        if (c < nk) issue(c, lds + c * S::STAGE);
    if (EARLY_TAIL && ktail) load_tail();
    if (EARLY_TAIL && nk < NST && ktail) store_tail(lds + (int)nk * S::STAGE);
    // (the count is of the newest loads: any others among them only make it wait longer)
    if (nk >= NST) wait_steps(std::integral_constant<int, NST - 1>());
    else wait_steps(std::integral_constant<int, 0>());
    __syncthreads();
    if (live && (!GROUPS || nk > 0)) {
#pragma unroll
        for (int g = 0; g < S::G; ++g) {
#pragma unroll
            for (int i = 0; i < S::FM; ++i) read_a(lds, g, i);
            read_b(lds, g, 0);
            read_b(lds, g, 1);
        }
    }
    int st = 0;
    int64_t c = 0;
    // while full k-steps are left to load: own loads of k-step c+1 landed, then
    // everyone's; every wave holds k-step c in registers
    for (; c + NST < nk; ++c) {
        wait_steps(std::integral_constant<int, NST - 2>());
        __syncthreads();
        const int st1 = st == NST - 1 ? 0 : st + 1;
        if (live)
            products(std::true_type(), std::true_type(), lds + st1 * S::STAGE, c + NST,
                     lds + st * S::STAGE);
        else
            issue(c + NST, lds + st * S::STAGE);
        st = st1;
    }
    // the rest: the element-wise k-step takes the stage that k-step nk - NST left
#pragma unroll 1
    for (; c < steps; ++c) {
        wait_steps(std::integral_constant<int, 0>());
        __syncthreads();
        const int st1 = st == NST - 1 ? 0 : st + 1;
        if (EARLY_TAIL && ktail && c + NST == nk) store_tail(lds + st * S::STAGE);
        if (live)
            products(std::false_type(), std::true_type(), lds + st1 * S::STAGE, 0, lds);
        st = st1;
    }
    if (EARLY_TAIL ? GROUPS && nk == 0 : ktail != 0) {
        if (!EARLY_TAIL) {
            load_tail();
            __syncthreads();             // every wave is done with LDS
            store_tail(lds);
            __syncthreads();
        }
        if (live) {
#pragma unroll
            for (int g = 0; g < S::G; ++g) {
                if (GROUPS && g * 8 >= ktail) break;
#pragma unroll
                for (int i = 0; i < S::FM; ++i) read_a(lds, g, i);
                read_b(lds, g, 0);
                read_b(lds, g, 1);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < S::FM; ++i)
#pragma unroll
                        for (int j = 0; j < S::FN; ++j)
                            acc[i][j] = E::mma(af[g][i][h], bf[g][h][j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
            }
            // what the products of the groups left out would add
            if (GROUPS && ktail <= BK - 8) {
#pragma unroll
                for (int i = 0; i < S::FM; ++i)
#pragma unroll
                    for (int j = 0; j < S::FN; ++j) acc[i][j] += acc4{0, 0, 0, 0};
            }
        }
    }

    if (!live) return;
    // Epilogue: lane holds column l16 and rows E::out_row(kq, 0..3) of each fragment.
    // The C loads of one fragment row go out together before its stores; on edge
    // tiles they read clamped addresses and the stores are tested.
    AS_GLOBAL T *__restrict__ C = (AS_GLOBAL T *)p.C;
    const int64_t ldc = p.ldc;
    const T alpha = (T)p.alpha, beta = (T)p.beta;
    const bool read_c = p.beta != 0.0;
    AS_GLOBAL T *Ct = C + m0 * ldc + n0;
    auto epilogue = [&](auto inside) {
        constexpr bool INTERIOR = decltype(inside)::value;
#pragma unroll
        for (int i = 0; i < S::FM; ++i) {
            T cv[S::FN][4];
            if (read_c) {
#pragma unroll
                for (int j = 0; j < S::FN; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        int64_t row = wm * S::WM + i * 16 + E::out_row(kq, r);
                        int64_t col = wn * S::WN + j * 16 + l16;
                        if (!INTERIOR) {
                            row = row < mrem ? row : mrem - 1;
                            col = col < nrem ? col : nrem - 1;
                            col = col < first_col ? first_col : col;
                        }
                        cv[j][r] = Ct[row * ldc + col];
                    }
            }
#pragma unroll
            for (int j = 0; j < S::FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t row = wm * S::WM + i * 16 + E::out_row(kq, r);
                    const int64_t col = wn * S::WN + j * 16 + l16;
                    if (!INTERIOR && (row >= mrem || col >= nrem || col < first_col)) continue;
                    AS_GLOBAL T *c = Ct + row * ldc + col;
                    *c = read_c ? scale_add(alpha, acc[i][j][r], beta, cv[j][r])
                                : alpha * acc[i][j][r];
                }
        }
    };
    if (mrem >= BM && nrem >= BN && first_col == 0) epilogue(std::true_type());
    else epilogue(std::false_type());
}

}  // namespace mgemm
