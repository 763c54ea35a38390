// One training step of the MLP cost model in two kernels: mlp_step_kernel takes a
// tile of training rows through the forward pass, the loss, the backward pass and
// that tile's share of every gradient without leaving LDS, and mlp_update_kernel
// adds the shares and applies Adam.
#pragma once

#include "tile_gemm.h"

namespace mgemm {

// The step kernel holds networks of at most STEP_MAX_IN inputs and STEP_MAX_HIDDEN
// hidden units (host_rules.h) in LDS: hidden width padded to HP = 64 (tiles of 64 rows)
// or 128 (32 rows), any number of outputs (in chunks of 64).
constexpr int STEP_CHUNK = 64;

struct MlpStepArgs {
    int I, H, O;
    int64_t B;                    // training rows
    const float *X, *T, *M;       // B x I, B x O, B x O
    const float *par;             // W1 b1 W2 b2 W3 b3
    float *planes;                // one gradient share per block, in parameter order
    int64_t plane;                // elements from one share to the next
    float *part;                  // 2 floats per block: sum of M, sum of M (y - t)^2
    int *step;                    // Adam step counter, advanced here (may be NULL)
};

template <int HP, int ROWS>
struct StepShape {
    static constexpr int SX = STEP_MAX_IN + 4;       // LDS row strides: rows 4 banks apart
    static constexpr int SH = HP + 4, SD = STEP_CHUNK + 4;
    static constexpr int X = ROWS * SX, H1 = ROWS * SH, H2 = ROWS * SH, D = ROWS * SD,
                         W2 = HP * SH, WB = STEP_CHUNK * SH;
    static constexpr int FLOATS = X + H1 + H2 + D + W2 + WB;
    static_assert(HP * SX <= WB && ROWS * SH <= WB, "W1 and dZ2 share the chunk's buffer");
    static_assert(FLOATS * 4 <= 160 * 1024, "LDS");
};

// acc[j] += A (16 x K) * B_j (K x 16) over LDS: element (m, k) of A at A[m*ams +
// k*aks], (k, n) of B_j at B[k*bks + n*bns + j*bstep].
template <int K, int NF>
__device__ __forceinline__ void step_mm(v4f (&acc)[NF], const float *A, int ams, int aks,
                                        const float *B, int bks, int bns, int bstep) {
    const int l16 = threadIdx.x & 15, kq = (threadIdx.x & 63) >> 4;
    const float *a = A + l16 * ams + kq * aks, *b = B + l16 * bns + kq * bks;
#pragma unroll
    for (int k = 0; k < K; k += 4) {
        const float av = a[k * aks];
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[j] = Elem<float>::mma(av, b[k * bks + j * bstep], acc[j]);
    }
}

// The gradient dW (frags: 16 rows from w0, NF x 16 columns from k0) of dZ^T A over K
// training rows, into the block's share (rows < nrows of ld columns; added where the
// block has taken a tile before), and with BIAS the row sums of dZ^T.
template <int K, int NF>
__device__ __forceinline__ void step_grad(const float *dZ, int zs, const float *A, int as, int w0,
                                          int k0, int nrows, int ld, float *gW, float *gb,
                                          bool bias, bool add) {
    const int l16 = threadIdx.x & 15, kq = (threadIdx.x & 63) >> 4;
    v4f acc[NF], ones = v4f{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[j] = v4f{0, 0, 0, 0};
    const float *a = dZ + w0 + l16 + kq * zs, *b = A + k0 + l16 + kq * as;
#pragma unroll
    for (int k = 0; k < K; k += 4) {
        const float av = a[k * zs];
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[j] = Elem<float>::mma(av, b[k * as + j * 16], acc[j]);
        if (bias) ones = Elem<float>::mma(av, 1.0f, ones);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = w0 + 4 * kq + r;
        if (row >= nrows) continue;
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int col = k0 + j * 16 + l16;
            if (col >= ld) continue;
            float *g = gW + (int64_t)row * ld + col;
            *g = add ? *g + acc[j][r] : acc[j][r];
        }
        if (bias && l16 == 0) gb[row] = add ? gb[row] + ones[r] : ones[r];
    }
}

// Eight waves take tiles of ROWS training rows in turn (grid: at most one block per
// compute unit).  Everything between the inputs and the gradient shares stays in LDS
// and registers; the shares are unscaled (the factor 2 / sum M needs every block) and
// rows past B and outputs past O have M = 0, so they add nothing.
//
// Bound: the matrix cores (about 8 products of ROWS x HP x 64 per 64 outputs, two
// waves per SIMD) and the latency between the barriers.  13600 rows x (6 -> 64 -> 64
// -> 247): 12 kernels with activations in memory took 231 us a step; this one takes
// 41 us (about 15 of them the products' matrix-core time) and the update 5.8.
template <int HP, int ROWS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
mlp_step_kernel(MlpStepArgs a) {
    typedef StepShape<HP, ROWS> S;
    __shared__ __attribute__((aligned(16))) float lds[S::FLOATS];
    __shared__ float red[16];
    float *sX = lds, *sH1 = sX + S::X, *sH2 = sH1 + S::H1, *sD = sH2 + S::H2, *sW2 = sD + S::D,
          *sWb = sW2 + S::W2;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I = a.I, H = a.H, O = a.O;
    const float *W1 = a.par, *b1 = W1 + (int64_t)H * I, *W2 = b1 + H, *b2 = W2 + (int64_t)H * H,
                *W3 = b2 + H, *b3 = W3 + (int64_t)O * H;
    float *gW1 = a.planes + blockIdx.x * a.plane, *gb1 = gW1 + (int64_t)H * I, *gW2 = gb1 + H,
          *gb2 = gW2 + (int64_t)H * H, *gW3 = gb2 + H, *gb3 = gW3 + (int64_t)O * H;
    if (a.step && blockIdx.x == 0 && tid == 0) *a.step += 1;   // read by the update kernel

    // fragment maps: ROWS x HP results (2 per wave), ROWS x 64 outputs, and the
    // gradients' 64 x HP, HP x HP and HP x 32
    constexpr int MR = ROWS / 16, GR = 8 / MR;
    const int mr = wave % MR, gr = wave / MR;
    constexpr int NY = 4 / GR;
    constexpr int N3 = HP / 32;
    constexpr int MH = HP / 16, GH = 8 / MH, N2 = MH / GH, N1 = 2 / GH;
    const int mh = wave % MH, gh = wave / MH;

    for (int e = tid; e < HP * HP; e += 512) {
        const int r = e / HP, c = e % HP;
        sW2[r * S::SH + c] = r < H && c < H ? W2[(int64_t)r * H + c] : 0.0f;
    }
    constexpr int CW = STEP_CHUNK * HP / 512;        // a thread's elements of a W3 chunk
    float w3[CW];
    auto load_w3 = [&](int o0) {
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int e = tid + 512 * j, r = e / HP, c = e % HP;
            w3[j] = o0 + r < O && c < H ? W3[(int64_t)(o0 + r) * H + c] : 0.0f;
        }
    };
    auto store_w3 = [&]() {
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int e = tid + 512 * j;
            sWb[e / HP * S::SH + e % HP] = w3[j];
        }
    };

    float cnt = 0.0f, sq = 0.0f;
    const int64_t tiles = (a.B + ROWS - 1) / ROWS;
    bool add = false;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t r0 = t * ROWS;
        __syncthreads();                             // the previous tile is done with LDS
        for (int e = tid; e < ROWS * STEP_MAX_IN; e += 512) {
            const int r = e / STEP_MAX_IN, c = e % STEP_MAX_IN;
            sX[r * S::SX + c] = r0 + r < a.B && c < I ? a.X[(r0 + r) * I + c] : 0.0f;
        }
        for (int e = tid; e < HP * STEP_MAX_IN; e += 512) {
            const int r = e / STEP_MAX_IN, c = e % STEP_MAX_IN;
            sWb[r * S::SX + c] = r < H && c < I ? W1[(int64_t)r * I + c] : 0.0f;
        }
        load_w3(0);
        __syncthreads();
        // a ROWS x HP layer's result: relu(acc + bias), zero past H
        auto store_relu = [&](const v4f (&acc)[2], const float *bias, float *dst) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int col = (gr * 2 + j) * 16 + l16;
                const float bv = col < H ? bias[col] : 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    dst[(mr * 16 + 4 * kq + r) * S::SH + col] = fmaxf(acc[j][r] + bv, 0.0f);
            }
        };
        {
            v4f acc[2] = {v4f{0, 0, 0, 0}, v4f{0, 0, 0, 0}};
            for (int k = 0; k < I; k += 4)           // columns past I are zero
                step_mm<4, 2>(acc, sX + mr * 16 * S::SX + k, S::SX, 1,
                              sWb + gr * 32 * S::SX + k, 1, S::SX, 16 * S::SX);
            store_relu(acc, b1, sH1);
        }
        __syncthreads();
        store_w3();
        {
            v4f acc[2] = {v4f{0, 0, 0, 0}, v4f{0, 0, 0, 0}};
            step_mm<HP, 2>(acc, sH1 + mr * 16 * S::SH, S::SH, 1, sW2 + gr * 32 * S::SH, 1, S::SH,
                           16 * S::SH);
            store_relu(acc, b2, sH2);
        }
        v4f dz2[2] = {v4f{0, 0, 0, 0}, v4f{0, 0, 0, 0}};
        for (int o0 = 0; o0 < O; o0 += STEP_CHUNK) {
            // this lane's targets and mask of the chunk, in flight during its product
            float tv[NY][4], mv[NY][4];
#pragma unroll
            for (int j = 0; j < NY; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int col = o0 + (gr * NY + j) * 16 + l16;
                    const int64_t row = r0 + mr * 16 + 4 * kq + r;
                    const bool in = col < O && row < a.B;
                    tv[j][r] = in ? a.T[row * O + col] : 0.0f;
                    mv[j][r] = in ? a.M[row * O + col] : 0.0f;
                }
            if (o0 + STEP_CHUNK < O) load_w3(o0 + STEP_CHUNK);
            __syncthreads();                         // H2 and the W3 chunk are in LDS
            {
                v4f acc[NY];
#pragma unroll
                for (int j = 0; j < NY; ++j) acc[j] = v4f{0, 0, 0, 0};
                step_mm<HP, NY>(acc, sH2 + mr * 16 * S::SH, S::SH, 1,
                                sWb + gr * NY * 16 * S::SH, 1, S::SH, 16 * S::SH);
#pragma unroll
                for (int j = 0; j < NY; ++j) {
                    const int c = (gr * NY + j) * 16 + l16;
                    const float bv = o0 + c < O ? b3[o0 + c] : 0.0f;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float d = acc[j][r] + bv - tv[j][r];
                        const float md = mv[j][r] * d;
                        const bool in = o0 + c < O && r0 + mr * 16 + 4 * kq + r < a.B;
                        sD[(mr * 16 + 4 * kq + r) * S::SD + c] = in ? md : 0.0f;
                        if (in) {
                            cnt += mv[j][r];
                            sq = fmaf(md, d, sq);
                        }
                    }
                }
            }
            __syncthreads();
            step_mm<STEP_CHUNK, 2>(dz2, sD + mr * 16 * S::SD, S::SD, 1, sWb + gr * 32, S::SH, 1, 16);
            step_grad<ROWS, N3>(sD, S::SD, sH2, S::SH, (wave & 3) * 16, (wave >> 2) * N3 * 16,
                                O - o0, H, gW3 + (int64_t)o0 * H, gb3 + o0, wave < 4, add);
            __syncthreads();                         // the chunk's readers are done
            if (o0 + STEP_CHUNK < O) store_w3();
        }
        // dZ2 = (D W3) where H2 > 0, in the chunk's buffer
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = (mr * 16 + 4 * kq + r) * S::SH + (gr * 2 + j) * 16 + l16;
                sWb[o] = sH2[o] > 0.0f ? dz2[j][r] : 0.0f;
            }
        __syncthreads();
        step_grad<ROWS, N2>(sWb, S::SH, sH1, S::SH, mh * 16, gh * N2 * 16, H, H, gW2, gb2, gh == 0,
                            add);
        {
            // dZ1 = (dZ2 W2) where H1 > 0, in H2's place
            v4f acc[2] = {v4f{0, 0, 0, 0}, v4f{0, 0, 0, 0}};
            step_mm<HP, 2>(acc, sWb + mr * 16 * S::SH, S::SH, 1, sW2 + gr * 32, S::SH, 1, 16);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int o = (mr * 16 + 4 * kq + r) * S::SH + (gr * 2 + j) * 16 + l16;
                    sH2[o] = sH1[o] > 0.0f ? acc[j][r] : 0.0f;
                }
        }
        __syncthreads();
        step_grad<ROWS, N1>(sH2, S::SH, sX, S::SX, mh * 16, gh * N1 * 16, H, I, gW1, gb1, gh == 0,
                            add);
        add = true;
    }
    // this block's sums, in a fixed order
    for (int off = 32; off > 0; off >>= 1) {
        cnt += __shfl_xor(cnt, off);
        sq += __shfl_xor(sq, off);
    }
    if (lane == 0) {
        red[wave] = cnt;
        red[8 + wave] = sq;
    }
    __syncthreads();
    if (tid == 0) {
        float c = 0.0f, s = 0.0f;
        for (int w = 0; w < 8; ++w) {
            c += red[w];
            s += red[8 + w];
        }
        a.part[2 * blockIdx.x] = c;
        a.part[2 * blockIdx.x + 1] = s;
    }
}

// g = 2 / sum M * (sum of the nb gradient shares, in a fixed order) for 32 parameters
// per block, 16 threads to a parameter, and with lr > 0 Adam's update of them (step
// number *step); block 0 also writes the loss sum M (y - t)^2 / sum M.
//
// Bound: the shares' bytes (nb x P x 4, 18 MB at 213 blocks x 20.6 k parameters) and the
// latency of two rounds of loads.  Eight threads to a parameter with one load in flight
// took 11.5 us, with eight 8.6; 16 threads, eight loads and shares on 256-byte
// boundaries 5.8.
constexpr int UPDATE_Z = 16, UPDATE_SHARE = 64;      // shares in multiples of this many elements

__global__ void __launch_bounds__(32 * UPDATE_Z)
mlp_update_kernel(const float *__restrict__ planes, int64_t plane, int nb, int64_t P,
                  const float *__restrict__ part, float *__restrict__ loss, float *__restrict__ grad,
                  float *__restrict__ p, float *__restrict__ m, float *__restrict__ v, float lr,
                  float b1, float b2, float eps, const int *step) {
    __shared__ float s_cnt[256], s_sq[256], s_g[32 * UPDATE_Z];
    const int tid = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * 32 + (tid & 31);
    float g = 0.0f;
    if (i < P)
        for (int z = tid >> 5; z < nb; z += 8 * UPDATE_Z) {
            float w[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int zj = z + UPDATE_Z * j;
                w[j] = planes[(int64_t)(zj < nb ? zj : z) * plane + i];
                if (zj >= nb) w[j] = 0.0f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) g += w[j];
        }
    s_g[tid] = g;
    if (tid < 256) {
        float cnt = 0.0f, sq = 0.0f;
        for (int z = tid; z < nb; z += 256) {
            cnt += part[2 * z];
            sq += part[2 * z + 1];
        }
        s_cnt[tid] = cnt;
        s_sq[tid] = sq;
    }
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) {
            s_cnt[tid] += s_cnt[tid + h];
            s_sq[tid] += s_sq[tid + h];
        }
        __syncthreads();
    }
    const float total = s_cnt[0] > 0.0f ? s_cnt[0] : 1.0f;
    if (blockIdx.x == 0 && tid == 0) *loss = s_sq[0] / total;
    if (tid >= 32 || i >= P) return;
    for (int z = 1; z < UPDATE_Z; ++z) g += s_g[tid + 32 * z];
    g *= 2.0f / total;
    grad[i] = g;
    if (!(lr > 0.0f)) return;
    const float t = (float)*step;
    const float bc1 = 1.0f - powf(b1, t);
    const float bc2 = 1.0f - powf(b2, t);
    const float mi = b1 * m[i] + (1.0f - b1) * g;
    const float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

}  // namespace mgemm
