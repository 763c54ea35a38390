// Modular-integer emulation of an FP64 GEMM on int8 matrix cores (Ozaki scheme
// II: Ozaki, Uchino, Imamura, "Ozaki Scheme II: A GEMM-oriented emulation of
// floating-point matrix multiplication using an integer modular technique", 2025).
//
// C = alpha*A*B + beta*C with FP64 A, B, C:
//  1. scale     e_i, f_j: exponents of the row / column maxima (shared with the
//               slice emulation); b = the operand width, the largest b <= 62 with
//               k 2^(2b) <= 2^123.
//  2. residues  A'_ip = trunc(A_ip 2^(b - e_i)) and B'_pj = trunc(B_pj 2^(b - f_j))
//               are integers below 2^b; their residues modulo the 16 moduli below,
//               in [-p/2, p/2), are stored as int8 planes (B transposed, so both
//               operands are k-contiguous).
//  3. products  one int8 GEMM per modulus on the matrix cores with exact int32
//               accumulation (in launches of at most 2^16 k, each adding its
//               residues to the previous ones), whose result modulo p is stored as
//               one byte per element.
//  4. combine   the Chinese remainder theorem gives the exact integer
//               C'_ij = sum_p A'_ip B'_pj from its 16 residues (|C'| <= 2^123, a
//               quarter of the moduli's product), which is rounded once to FP64,
//               scaled by 2^(e_i + f_j - 2b) and the epilogue alpha*v + beta*C
//               applied.
//
// Against the slice emulation with int8 slices (36 slice-pair products of the
// same operand width), this needs 16 products of the full width, each a plain
// int8 GEMM.
#include <limits.h>
#include <math.h>

#include "mgemm_internal.h"

namespace mgemm {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Pairwise coprime moduli, the largest such set below 2^8: product > 2^125.37.

// The moduli as compile-time constants for the device (t is unrolled), so the
// residues use constant-divisor arithmetic.
__host__ __device__ constexpr int modulus(int t) {
    return t == 0 ? 256 : t == 1 ? 255 : t == 2 ? 253 : t == 3 ? 251 : t == 4 ? 247 :
           t == 5 ? 241 : t == 6 ? 239 : t == 7 ? 233 : t == 8 ? 229 : t == 9 ? 227 :
           t == 10 ? 223 : t == 11 ? 217 : t == 12 ? 211 : t == 13 ? 199 : t == 14 ? 197 : 193;
}
// 2^e mod p_t
__host__ __device__ constexpr int pow2_mod(int t, int e) {
    return (int)(((uint64_t)1 << e) % (uint64_t)modulus(t));
}
__constant__ int kModuliDev[CRT_MODULI] = {modulus(0),  modulus(1),  modulus(2),  modulus(3),
                                           modulus(4),  modulus(5),  modulus(6),  modulus(7),
                                           modulus(8),  modulus(9),  modulus(10), modulus(11),
                                           modulus(12), modulus(13), modulus(14), modulus(15)};

// ---------------------------------------------------------------------------
// 2. Residues.
// ---------------------------------------------------------------------------
// Residues of integers a (|a| < 2^62, held exactly in doubles) modulo each p, as int8
// in [-p/2, p/2).  a + 2^63 is a 64-bit word of eight bytes y_i, so a = sum_i y_i c_i +
// K (mod p) with c_i = 2^(8i) mod p and K = -2^63 mod p: two byte dot products with K
// as their start.  The sum s stays below 2^19.3, and with h = p / 2 rounded down the
// quotient floor((s + h) / p) is the high word of 16 (s + h) times ceil(2^28 / p), both
// factors below 2^24 (exact for every s + h < 2^20: the factor's excess adds less than
// 2^-8 < 1 / p).  Five instructions per residue, where 16-bit digits with 32-bit
// products and a 32-bit reduction took about twelve.
__host__ __device__ constexpr uint32_t byte_consts(int t, int e0) {
    return (uint32_t)pow2_mod(t, e0) | (uint32_t)pow2_mod(t, e0 + 8) << 8 |
           (uint32_t)pow2_mod(t, e0 + 16) << 16 | (uint32_t)pow2_mod(t, e0 + 24) << 24;
}

// The bytes of a + 2^63 as two words (lo, hi).
struct Bytes8 {
    uint32_t lo, hi;
};

__device__ inline Bytes8 bytes_of(double a) {
    const double hi = floor(a * 0x1p-32);
    return {(uint32_t)(a - hi * 0x1p32), (uint32_t)(int)hi ^ 0x80000000u};
}

// Residue t of the integer with bytes y, in the low byte.
template <int t>
__device__ inline uint32_t residue(Bytes8 y) {
    constexpr int p = modulus(t), h = p / 2;
    constexpr uint32_t K = (uint32_t)((p - pow2_mod(t, 63)) % p);
    constexpr uint32_t M = ((1u << 28) + p - 1) / p;
    static_assert(M < (1u << 24) && 8 * 255 * 255 + 2 * 256 < (1 << 20), "24-bit quotient");
    const uint32_t s = __builtin_amdgcn_udot4(
        y.hi, byte_consts(t, 32), __builtin_amdgcn_udot4(y.lo, byte_consts(t, 0), K, false), false);
    const uint32_t u = (s << 4) + 16u * (uint32_t)h;
    const uint32_t q = (uint32_t)(((uint64_t)(u & 0xFFFFFFu) * M) >> 32);
    return s - (uint32_t)__mul24((int)q, p);
}

// The low bytes of four words as one word.
__device__ inline uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
    const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
    return ab | cd << 16;
}

// Residues t.. of N integers (N a multiple of 4), N / 4 words per modulus, each handed
// to store(modulus, words).
template <int N, int t = 0, typename F>
__device__ inline void residues_each(const Bytes8 (&y)[N], F store) {
    uint32_t w[N / 4];
#pragma unroll
    for (int i = 0; i < N / 4; ++i)
        w[i] = pack4(residue<t>(y[4 * i]), residue<t>(y[4 * i + 1]), residue<t>(y[4 * i + 2]),
                     residue<t>(y[4 * i + 3]));
    store(t, w);
    if constexpr (t + 1 < CRT_MODULI) residues_each<N, t + 1>(y, store);
}

// Block per 8 rows x 256 k of A, thread per (row, 8 consecutive k): a wave writes runs
// of 512 bytes (8 rows of one chunk), and neighbouring blocks read on along the rows
// (blocks of 32 rows x 64 k, one memory channel under all rows of a power-of-two
// leading dimension, took 184 us at 4096^2 instead of 135).  Rows >= m and k >= k give
// zeros.
__global__ void __launch_bounds__(256)
crt_residue_a_kernel(const double *__restrict__ A, int64_t m, int64_t k, int64_t lda,
                     const int *__restrict__ e, int bits, int8_t *__restrict__ Q, int64_t mp,
                     int64_t kp) {
    const int tid = threadIdx.x;
    const int64_t chunk = (int64_t)blockIdx.x * 4 + (tid >> 6);
    const int64_t p0 = chunk * CRT_KSTEP + (tid & 7) * 8;
    if (p0 >= kp) return;
    const int64_t plane = mp * kp;
    for (int64_t i = (int64_t)blockIdx.y * 8 + ((tid >> 3) & 7); i < mp; i += (int64_t)gridDim.y * 8) {
        const int ex = i < m ? e[i] : 0;
        Bytes8 y[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int64_t p = p0 + v;
            y[v] = bytes_of((i < m && p < k) ? trunc(ldexp(A[i * lda + p], bits - ex)) : 0.0);
        }
        int8_t *dst = Q + (chunk * mp + i) * CRT_KSTEP + (tid & 7) * 8;
        residues_each(y, [&](int t, const uint32_t (&w)[2]) {
            *(uint2 *)(dst + t * plane) = make_uint2(w[0], w[1]);
        });
    }
}

// 64 (k) x 64 (n) tile of B through LDS; thread (column j, 16 consecutive k) ->
// the residues of column j, stored k-contiguous.
__global__ void __launch_bounds__(256)
crt_residue_b_kernel(const double *__restrict__ B, int64_t k, int64_t n, int64_t ldb,
                     const int *__restrict__ fexp, int bits, int8_t *__restrict__ Q, int64_t np,
                     int64_t kp) {
    __shared__ double tile[64][65];
    const int tid = threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.x * 64;
    const int64_t p0 = (int64_t)blockIdx.y * 64;
    for (int idx = tid; idx < 64 * 64; idx += 256) {
        const int pr = idx >> 6, jc = idx & 63;
        const int64_t p = p0 + pr, j = j0 + jc;
        tile[pr][jc] = (p < k && j < n) ? B[p * ldb + j] : 0.0;
    }
    __syncthreads();
    const int jc = tid >> 2;
    const int pg = (tid & 3) * 16;
    const int64_t j = j0 + jc;
    const int fe = j < n ? fexp[j] : INT_MIN;
    const int ex = fe == INT_MIN ? 0 : fe;
    Bytes8 y[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) y[v] = bytes_of(trunc(ldexp(tile[pg + v][jc], bits - ex)));
    const int64_t plane = np * kp;
    int8_t *dst = Q + p0 * np + j * CRT_KSTEP + pg;
    residues_each(y, [&](int t, const uint32_t (&w)[4]) {
        *(u32x4 *)(dst + t * plane) = u32x4{w[0], w[1], w[2], w[3]};
    });
}

// ---------------------------------------------------------------------------
// 3. One int8 GEMM per modulus.
// ---------------------------------------------------------------------------
// Work-group: WGM x WGN waves own a 256 x 256 tile of C for one modulus; each
// wave a (256/WGM) x (256/WGN) block as 32x32 accumulators of the 32x32x32 int8
// MFMA.  A stage holds 64 k of the tile's 256 A rows and 256 B columns; the
// stages are filled by direct global->LDS loads NST-1 stages ahead, and every
// fragment register is refilled from the next stage right after its last use.
// Operands are zero-padded to whole tiles and stages, so no load or store needs
// a bounds test.  A plane holds its chunks of 64 k one after another, each with the 64
// bytes of all rows in turn, so a stage's 256 rows are one run of 16 KB: with rows of
// kp bytes every 128-byte line was asked for twice, half each time (4096^3: 1.43e8 L2
// requests and 1207 us, 7.3e7 and 1140 us in chunks).
constexpr int G_KS = CRT_KSTEP;                 // k per stage
constexpr int G_PASS = (1 << 16) / G_KS;        // stages per launch: |acc| < 2^16 * 2^14

// LDS layout of one stage: 256 A rows then 256 B rows of 64 k (4 units of 16 B).
//  PADDED:   rows of 5 units (the fifth a copy, never read); four stages.
//  SWIZZLED: rows of 4 units, logical unit c of row r stored at c ^ sw(r) with
//            sw(r) = (r >> 2) & 3; five stages in the same space.
// Both keep the fragment reads free of bank conflicts (SQ_LDS_BANK_CONFLICT reads
// 0 for either; of the XOR patterns tried, (r >> 1) & 3 or ((r >> 1) ^ (r >> 3)) & 3
// conflict on half of the LDS cycles, r & 3 on three quarters).
template <bool SWZ> struct StageLayout {
    static constexpr int ROW = SWZ ? 4 : 5;                 // units per LDS row
    static constexpr int AUNITS = CRT_TILE * ROW;           // A part of a stage
    static constexpr int STAGE = 2 * AUNITS;                // units per stage
    static constexpr int NST = SWZ ? 5 : 4;                 // stages
    static_assert(AUNITS % 64 == 0, "a wave's loads lie in one operand");
    static_assert(NST * STAGE * 16 <= 163840, "LDS");
    __device__ static int sw(int r) { return SWZ ? (r >> 2) & 3 : 0; }
};

struct CrtGemmArgs {
    const int8_t *QA;
    const int8_t *QB;
    uint8_t *R;
    int64_t plane_a, plane_b, plane_r;
    int64_t np;
    int tiles_m, tiles_n;
    int ch0, ch1;          // stages [ch0, ch1) of this pass (at most 2^16 k)
    int accumulate;        // add the previous passes' residues already in R
};

// Bound: the matrix cores and LDS together (98 KB of fragment reads and 32 KB of
// loads per 1030 cycles of products), at the clock their power leaves.  At 4096^3 the
// epilogue counted as much as the k-loop while it divided twice per element and stored
// single bytes: see the figures there.
// 32x32 accumulator element r of lane l: row (here a column of C) 8(r/4) + 4(l/32) +
// r%4, column (here a row of C) l%32.
template <int WGM, int WGN, bool SWZ>
__global__ void __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(WGM * WGN / 4)))
crt_gemm_kernel(CrtGemmArgs a) {
    typedef StageLayout<SWZ> L;
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WTM = CRT_TILE / WGM, WTN = CRT_TILE / WGN;   // wave block
    constexpr int FM = WTM / 32, FN = WTN / 32;                 // accumulators per wave
    constexpr int LOADS = L::STAGE / NT;                        // loads per lane per stage
    constexpr int NST = L::NST;
    static_assert(L::STAGE % NT == 0, "load split");
    __shared__ u32x4 lds[NST * L::STAGE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    // work-group -> (modulus, tile): the moduli one after another, each walked as
    // one GEMM's tiles (XCD-aware, grouped rows)
    const int tiles = a.tiles_m * a.tiles_n;
    int lid = blockIdx.x;
    {
        const int full = (int)(gridDim.x / 8) * 8;
        if (lid < full) lid = (lid % 8) * (full / 8) + lid / 8;
    }
    const int t = lid / tiles;
    int tm, tn;
    tile_of_block(lid - t * tiles, 0, a.tiles_m, a.tiles_n, tm, tn);
    const int p = kModuliDev[t];
    const int8_t *qa = a.QA + t * a.plane_a + (int64_t)tm * CRT_TILE * G_KS;
    const int8_t *qb = a.QB + t * a.plane_b + (int64_t)tn * CRT_TILE * G_KS;
    // bytes from one chunk of 64 k to the next
    const int64_t chunk_a = (int64_t)a.tiles_m * CRT_TILE * G_KS,
                  chunk_b = (int64_t)a.tiles_n * CRT_TILE * G_KS;

    // per-lane source offsets: LDS unit u of a stage holds row r, logical unit c
    uint32_t off[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int u = i * NT + wave * 64 + lane;
        const int v = u < L::AUNITS ? u : u - L::AUNITS;
        const int r = v / L::ROW, pu = v % L::ROW;
        const int c = SWZ ? (pu ^ L::sw(r)) : (pu < 4 ? pu : 3);
        off[i] = (uint32_t)r * (uint32_t)G_KS + (uint32_t)c * 16u;
    }
    // load instruction i of chunk `chunk` into stage st
    auto issue_one = [&](int i, int chunk, int st) {
        const int first = i * NT + wave * 64;                     // uniform per wave
        const bool in_a = (i + 1) * NT <= L::AUNITS || (i * NT < L::AUNITS && first < L::AUNITS);
        const int8_t *src = (in_a ? qa + chunk * chunk_a : qb + chunk * chunk_b) + off[i];
        __builtin_amdgcn_global_load_lds((const void *)src,
                                         (__attribute__((address_space(3))) void *)(lds + st * L::STAGE + first),
                                         16, 0, 0);
    };
    auto issue = [&](int chunk, int st) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) issue_one(i, chunk, st);
    };

    v16i acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = v16i{};

    // fragment rows of this lane: the swizzle is the same for rows 32 apart
    const int ra = wm * WTM + (lane & 31), rb = wn * WTN + (lane & 31);
    int a_unit[2], b_unit[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int c = kk * 2 + (lane >> 5);
        a_unit[kk] = ra * L::ROW + (c ^ L::sw(ra));
        b_unit[kk] = L::AUNITS + rb * L::ROW + (c ^ L::sw(rb));
    }
    v4i fa[2][FM], fb[2][FN];
    auto read_a = [&](const u32x4 *st, int kk, int mt) {
        fa[kk][mt] = __builtin_bit_cast(v4i, st[a_unit[kk] + mt * 32 * L::ROW]);
    };
    auto read_b = [&](const u32x4 *st, int kk, int nt) {
        fb[kk][nt] = __builtin_bit_cast(v4i, st[b_unit[kk] + nt * 32 * L::ROW]);
    };
    // products of one stage; each fragment is refilled from the next stage right
    // after its last use (past the last stage the refills read a stale stage and
    // are never used)
    // The stage's loads (chunk lc into stage ls) are spread over the products, one
    // after every 2*FM/LOADS fragment rows, so that the memory pipeline takes them
    // a few at a time instead of all waves queueing every load at the barrier.
    auto products = [&](const u32x4 *nst, int lc, int ls) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
            for (int mt = 0; mt < FM; ++mt) {
#pragma unroll
                for (int nt = 0; nt < FN; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[kk][nt], fa[kk][mt],
                                                                         acc[mt][nt], 0, 0, 0);
                read_a(nst, kk, mt);
                constexpr int every = 2 * FM / LOADS > 0 ? 2 * FM / LOADS : 1;
                static_assert((LOADS - 1) * every < 2 * FM, "every load gets a slot");
                const int slot = kk * FM + mt;
                if (slot % every == 0 && slot / every < LOADS) issue_one(slot / every, lc, ls);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int nt = 0; nt < FN; ++nt) read_b(nst, kk, nt);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // stages of this pass, counted from its first.  Chunks 0..NST-2 in flight;
    // wait for chunk 0 (the loads of NST-2 chunks may remain)
    qa += (int64_t)a.ch0 * chunk_a;
    qb += (int64_t)a.ch0 * chunk_b;
    const int nst = a.ch1 - a.ch0;
#pragma unroll
    for (int c = 0; c < NST - 1; ++c) issue(c < nst ? c : nst - 1, c);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * LOADS));
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int mt = 0; mt < FM; ++mt) read_a(lds, kk, mt);
#pragma unroll
        for (int nt = 0; nt < FN; ++nt) read_b(lds, kk, nt);
    }
    int st = 0;                                   // stage of chunk c
    for (int c = 0; c < nst; ++c) {
        // chunk c+1 has landed (the loads of NST-3 later chunks may remain)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 3) * LOADS));
        __syncthreads();
        const int st1 = st + 1 == NST ? 0 : st + 1;
        const int stn = st == 0 ? NST - 1 : st - 1;    // stage of chunk c-1
        // chunk c+NST-1 into the stage of chunk c-1 (past the end: the last chunk
        // again, in bounds and never used)
        products(lds + st1 * L::STAGE, c + NST - 1 < nst ? c + NST - 1 : nst - 1, stn);
        st = st1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));       // no load lands after this point

    // Residues modulo p, packed and stored through LDS.  The products were formed
    // transposed (columns of B as the MFMA's rows), so elements 4g..4g+3 of a lane are
    // four neighbouring columns of one row: one 32-bit word, 32 words per lane, and the
    // tile's rows leave in whole 256-byte runs.
    const uint32_t M = (uint32_t)(0x100000000ull / (uint32_t)p);   // uniform
    const uint32_t bias = (uint32_t)p * (uint32_t)((1 << 30) / p + 1);
    constexpr int ROWB = CRT_TILE + 8;                 // LDS row stride (bytes)
    static_assert(CRT_TILE * ROWB <= NST * L::STAGE * 16, "the tile's residues fit the stages");
    uint8_t *R = a.R + t * a.plane_r + (int64_t)tm * CRT_TILE * a.np + (int64_t)tn * CRT_TILE;
    uint8_t *tile = (uint8_t *)lds;
    __syncthreads();                                   // every wave is done with the stages
#pragma unroll
    for (int mt = 0; mt < FM; ++mt)
#pragma unroll
        for (int nt = 0; nt < FN; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int row = wm * WTM + mt * 32 + (lane & 31);
                const int col = wn * WTN + nt * 32 + 8 * g + 4 * (lane >> 5);
                uint32_t old = 0;
                if (a.accumulate) old = *(const uint32_t *)(R + (int64_t)row * a.np + col);
                uint32_t word = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // |acc| <= 2^30, so u < 2^31 + 256; the quotient estimate is the
                    // floor of u / p or one less
                    const uint32_t u = (uint32_t)acc[mt][nt][4 * g + r] + bias;
                    uint32_t v = u - __umulhi(u, M) * (uint32_t)p;
                    v = min(v, v - (uint32_t)p);
                    if (a.accumulate) {
                        v += (old >> (8 * r)) & 0xFFu;
                        v = min(v, v - (uint32_t)p);
                    }
                    word |= v << (8 * r);
                }
                *(uint32_t *)(tile + row * ROWB + col) = word;
            }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CRT_TILE * CRT_TILE / 8 / NT; ++i) {
        const int u = i * NT + tid, row = u / (CRT_TILE / 8), c = u % (CRT_TILE / 8) * 8;
        *(uint64_t *)(R + (int64_t)row * a.np + c) = *(const uint64_t *)(tile + row * ROWB + c);
    }
}

// ---------------------------------------------------------------------------
// 4. Chinese-remainder reconstruction, one rounding, epilogue.
// ---------------------------------------------------------------------------
// With P the moduli's product, M_t = P / p_t and W_t = M_t (M_t^-1 mod p_t) < P,
// S = sum_t r_t W_t is congruent to C' modulo P; q = round(S / P) is found from
// the upper digits of S in FP64 (|C'| <= P/4 keeps S/P within 1/4 of q, far above
// the estimate's error), and C' = S - q P is computed modulo 2^128, which is exact
// because |C'| < 2^127.
struct CrtReconArgs {
    uint32_t w[CRT_MODULI / 4][16]; // byte j of W_4g..W_4g+3, four to a word
    double digit[4];                // 2^(64 + 16 i) / P
    uint32_t pl[4];                 // P as four 32-bit limbs
};

// Signed 128-bit integer (hi, lo) -> FP64, rounded to nearest even.
__device__ inline double i128_to_double(uint64_t hi, uint64_t lo) {
    const bool neg = (int64_t)hi < 0;
    if (neg) {
        lo = ~lo + 1;
        hi = ~hi + (lo == 0 ? 1 : 0);
    }
    double v;
    if (hi == 0) {
        v = (double)lo;                            // one rounding of an exact sum
    } else {
        const int lz = __clzll((long long)hi);     // 0..63
        const int drop = 64 - lz;                  // bits below the top 64
        const uint64_t top = lz == 0 ? hi : (hi << lz) | (lo >> drop);
        const uint64_t rest = lz == 0 ? lo : lo << lz;
        // a nonzero remainder below the top 64 bits turns an exact half into
        // "above half"; it cannot change any other rounding decision
        v = ldexp((double)(top | (rest != 0 ? 1 : 0)), drop);
    }
    return neg ? -v : v;
}

// C' of one element from its 16 residues, four to a word (r[g] holds t = 4g..4g+3).
// Byte j of the moduli's weights forms sum_t r_t W_t[j] < 2^20 by four byte dot
// products; pairs of bytes make digits of 16 bits (below 2^29), whose upper four give
// S / P (the lower four are below 2^-45 of P), and pairs of digits 32-bit limbs.
__device__ inline double crt_value(const uint32_t (&r)[CRT_MODULI / 4], const CrtReconArgs &rc) {
    uint32_t d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        uint32_t s0 = 0, s1 = 0;
#pragma unroll
        for (int g = 0; g < CRT_MODULI / 4; ++g) {
            s0 = __builtin_amdgcn_udot4(r[g], rc.w[g][2 * i], s0, false);
            s1 = __builtin_amdgcn_udot4(r[g], rc.w[g][2 * i + 1], s1, false);
        }
        d[i] = s0 + (s1 << 8);
    }
    double qf = (double)d[4] * rc.digit[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) qf = fma((double)d[4 + i], rc.digit[i], qf);
    const uint32_t q = (uint32_t)rint(qf);         // < 16 * 256
    // limbs below 2^46, minus q P limb by limb (q P_l < 2^44); carries propagate as
    // signed values, everything modulo 2^128
    auto limb = [&](int l) {
        return (int64_t)((uint64_t)d[2 * l] + ((uint64_t)d[2 * l + 1] << 16)) -
               (int64_t)((uint64_t)q * rc.pl[l]);
    };
    const int64_t d0 = limb(0);
    const int64_t d1 = limb(1) + (d0 >> 32);
    const int64_t d2 = limb(2) + (d1 >> 32);
    const int64_t d3 = limb(3) + (d2 >> 32);
    const uint64_t lo = ((uint64_t)(uint32_t)d1 << 32) | (uint32_t)d0;
    const uint64_t hi = ((uint64_t)(uint32_t)d3 << 32) | (uint32_t)d2;
    return i128_to_double(hi, lo);
}

// Bytes 0..3 of four words a_t, as four words of one byte of each.
__device__ inline void transpose4(const uint32_t (&a)[4], uint32_t (&c)[4]) {
    const uint32_t l01 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u);
    const uint32_t h01 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
    const uint32_t l23 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u);
    const uint32_t h23 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    c[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u);
    c[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u);
    c[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u);
    c[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
}

// A work-group takes 16 rows x 128 columns of C at a time, a thread 8 consecutive
// elements of a row: one 8-byte load per modulus.  The values change lanes through LDS
// (element v of a row's thread c at v RECON_V + c: every access spread over the banks),
// so that a wave reads and stores runs of 64 elements of C.
//
// Bound: about 130 integer and FP64 instructions per element, and 24 bytes.  4096^2: 118
// us; 153 with a thread storing its eight elements itself (64 lanes, 64 lines) and a
// 64-bit division per thread for its row.
constexpr int RECON_ROWS = 16, RECON_COLS = 128;
constexpr int RECON_V = 24, RECON_ROW = 8 * RECON_V + 16;

__global__ void __launch_bounds__(256)
crt_reconstruct_kernel(const uint8_t *__restrict__ R, int64_t plane_r, int64_t np,
                       const int *__restrict__ e, const int *__restrict__ fexp, int two_bits,
                       double *__restrict__ C, int64_t m, int64_t n, int64_t ldc, double alpha,
                       double beta, CrtReconArgs rc) {
    __shared__ double vals[RECON_ROWS * RECON_ROW];
    const int tid = (int)threadIdx.x, row = tid >> 4, c8 = tid & 15;
    const int wave = tid >> 6, lane = tid & 63;
    const int64_t cols0 = (int64_t)blockIdx.x * RECON_COLS, j0 = cols0 + 8 * c8;
    for (int64_t i0 = (int64_t)blockIdx.y * RECON_ROWS; i0 < m; i0 += (int64_t)gridDim.y * RECON_ROWS) {
        const int64_t i = i0 + row;
        if (i < m && j0 < n) {
            // residues of element v: rr[v][g] holds t = 4g..4g+3
            uint32_t rr[8][CRT_MODULI / 4];
#pragma unroll
            for (int g = 0; g < CRT_MODULI / 4; ++g) {
                uint32_t lo[4], hi[4], cl[4], ch[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const uint2 w = *(const uint2 *)(R + (4 * g + x) * plane_r + i * np + j0);
                    lo[x] = w.x;
                    hi[x] = w.y;
                }
                transpose4(lo, cl);
                transpose4(hi, ch);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    rr[x][g] = cl[x];
                    rr[4 + x][g] = ch[x];
                }
            }
            const int ei = e[i];
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const int fe = j0 + v < n ? fexp[j0 + v] : 0;
                const double cv = crt_value(rr[v], rc);
                vals[row * RECON_ROW + v * RECON_V + c8] =
                    ldexp(cv, ei + (fe == INT_MIN ? 0 : fe) - two_bits);
            }
        }
        __syncthreads();
        // a wave's four rows, 64 columns at a time
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = wave * 4 + (q >> 1), j = (q & 1) * 64 + lane;
            if (i0 + r < m && cols0 + j < n) {
                const double val = vals[r * RECON_ROW + (j & 7) * RECON_V + (j >> 3)];
                double *c = C + (i0 + r) * ldc + cols0 + j;
                if (beta == 0.0) {
                    *c = alpha * val;
                } else {
#pragma clang fp contract(off)
                    *c = alpha * val + beta * *c;
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
namespace {

struct CrtTables {
    CrtReconArgs rc;
    CrtTables() {
        typedef unsigned __int128 u128;
        u128 P = 1;
        for (int t = 0; t < CRT_MODULI; ++t) P *= (u128)modulus(t);
        for (int t = 0; t < CRT_MODULI; ++t) {
            const int p = modulus(t);
            const u128 M = P / (u128)p;
            // inverse of M mod p by the extended Euclidean algorithm
            long long r0 = (long long)(M % (u128)p), r1 = p, s0 = 1, s1 = 0;
            while (r1 != 0) {
                const long long qq = r0 / r1;
                long long tmp = r0 - qq * r1; r0 = r1; r1 = tmp;
                tmp = s0 - qq * s1; s0 = s1; s1 = tmp;
            }
            const long long inv = ((s0 % p) + p) % p;       // r0 == 1: coprime moduli
            const u128 W = M * (u128)inv;                    // < P: inv < p
            for (int j = 0; j < 16; ++j) {
                uint32_t &w = rc.w[t / 4][j];
                if (t % 4 == 0) w = 0;
                w |= (uint32_t)(uint8_t)(W >> (8 * j)) << (8 * (t % 4));
            }
        }
        for (int i = 0; i < 4; ++i) rc.digit[i] = ldexp(1.0, 64 + 16 * i) / (double)P;
        for (int l = 0; l < 4; ++l) rc.pl[l] = (uint32_t)(P >> (32 * l));
    }
};

const CrtTables &tables() {
    static const CrtTables tb;
    return tb;
}

}  // namespace

// The operand width b: the largest b <= 62 with k 2^(2b) <= 2^123, i.e.
// k <= 2^(123 - 2b) (at least 1).
int crt_operand_bits(int64_t k) {
    int b = 62;
    for (; b > 1; --b) {
        const int sh = 123 - 2 * b;
        if (sh >= 0 && (sh >= 63 || k <= ((int64_t)1 << sh))) break;
    }
    return b;
}

hipError_t crt_residues(const GemmArgs &g, hipStream_t s, const int *e, const int *fexp, int bits,
                        int8_t *QA, int8_t *QB, int64_t mp, int64_t np, int64_t kp) {
    {
        const unsigned gy = (unsigned)(mp / 8 < 65535 ? mp / 8 : 65535);
        hipLaunchKernelGGL(crt_residue_a_kernel, dim3((unsigned)((kp + 255) / 256), gy), dim3(256), 0,
                           s, (const double *)g.A, g.m, g.k, g.lda, e, bits, QA, mp, kp);
        hipLaunchKernelGGL(crt_residue_b_kernel, dim3((unsigned)(np / 64), (unsigned)(kp / 64)),
                           dim3(256), 0, s, (const double *)g.B, g.k, g.n, g.ldb, fexp, bits, QB,
                           np, kp);
    }
    return hipGetLastError();
}

hipError_t crt_products(const GemmArgs &g, hipStream_t s, const int *e, const int *fexp, int bits,
                        const int8_t *QA, const int8_t *QB, uint8_t *R, int64_t mp, int64_t np,
                        int64_t kp) {
    const CrtTables &tb = tables();
    {
        CrtGemmArgs ga;
        ga.QA = QA;
        ga.QB = QB;
        ga.R = R;
        ga.plane_a = mp * kp;
        ga.plane_b = np * kp;
        ga.plane_r = mp * np;
        ga.np = np;
        ga.tiles_m = (int)(mp / CRT_TILE);
        ga.tiles_n = (int)(np / CRT_TILE);
        const int64_t nstages = kp / CRT_KSTEP;
        const int64_t blocks = (int64_t)ga.tiles_m * ga.tiles_n * CRT_MODULI;
        // passes of at most 2^16 k keep the int32 sums exact; later passes add
        // their residues to the stored ones
        for (int64_t c0 = 0; c0 < nstages; c0 += G_PASS) {
            ga.ch0 = (int)c0;
            ga.ch1 = (int)(c0 + G_PASS < nstages ? c0 + G_PASS : nstages);
            ga.accumulate = c0 > 0;
            // 8 waves of 128 x 64 (two per SIMD) measured faster than 4 waves of
            // 128 x 128 (one per SIMD), which spend more time exposed at the barrier
            // (the swizzled five-stage layout measured 3 % faster than the padded
            // four-stage one)
            hipLaunchKernelGGL((crt_gemm_kernel<2, 4, true>), dim3((unsigned)blocks), dim3(512), 0, s, ga);
        }
    }
    {
        const int64_t rows = (g.m + RECON_ROWS - 1) / RECON_ROWS;
        hipLaunchKernelGGL(crt_reconstruct_kernel,
                           dim3((unsigned)((g.n + RECON_COLS - 1) / RECON_COLS),
                                (unsigned)(rows < 65535 ? rows : 65535)),
                           dim3(256), 0, s,
                           (const uint8_t *)R, mp * np, np, e, fexp, 2 * bits, (double *)g.C, g.m,
                           g.n, g.ldc, g.alpha, g.beta, tb.rc);
    }
    return hipGetLastError();
}

}  // namespace mgemm
