// The two-layer perceptron: its first layer forward, and the end of a training step (all gradients and the update).
//
// A step of 64 samples moves about 9 MB and computes 100 Mflop: every launch is latency, a chain of loads of about 1 us each.
// The step therefore takes two launches: the head, and gradients + update, whose workgroups go on to multiply the weights they have
// just updated with the next batch (the first step's first layer, and large batches, take a launch of their own).  The batch is never copied: rows of the pool
// are read through the selection list.  The first layer's partial sums are added by the head (which pools `positions` rows
// per sample anyway), and a gradient goes from the accumulators straight into the momentum and the parameter.
// Pass of 4 steps of 64 with 128 hidden units and a pool of 256: 272 us with nine launches a step, 97 with three, 89 with two.
#include "kernels.h"

// Four consecutive floats of a row of `cols`, from column c; past the end, or without 16-byte alignment, element by element.
__device__ __forceinline__ f32x4 load_cols4(const float* __restrict__ row, int c, int cols, bool vec) {
    if (vec && c + 3 < cols) return *reinterpret_cast<const f32x4*>(row + c);
    f32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = c + j < cols ? row[c + j] : 0.f;
    return v;
}

// part[b][z][h] = sum over the z-th part of the inputs of x[row b][i] W[h][i].  A workgroup owns 16 samples x 16 hidden units and
// one part; its four waves take a quarter of the part each and meet in LDS.  Lane l supplies row l % 16 of both factors and, in a
// step of 16 inputs, inputs 4 (l / 16) .. + 3, so that both are 16-byte loads.  The loads of STEPS steps are in flight together
// (3072 inputs over 32 waves are six steps, a part of 256 over its four waves four: one round trip to memory).
template <int STEPS>
__global__ __launch_bounds__(256) void mlp_fc1_kernel(const float* __restrict__ x, BatchRows rows, const float* __restrict__ W, int B, int hid, int K,
                                                      int k_wave, float* __restrict__ part, int x_vec, int w_vec) {
    __shared__ f32x4 red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.x * 16, n0 = blockIdx.y * 16;
    const int k_begin = (blockIdx.z * 4 + wave) * k_wave, k_end = min(K, k_begin + k_wave);
    const int m = min(m0 + r, B - 1);   // rows past the batch repeat its last one and are not stored
    const float* xr = x + pool_row(rows, m) * K;
    const float* wr = W + (int64_t)(n0 + r) * K;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = k_begin; k0 < k_end; k0 += 16 * STEPS) {
        f32x4 a[STEPS], b[STEPS];
        if (x_vec && w_vec && k0 + 16 * STEPS <= k_end) {
#pragma unroll
            for (int u = 0; u < STEPS; ++u) {
                a[u] = *reinterpret_cast<const f32x4*>(xr + k0 + 16 * u + 4 * g);
                b[u] = *reinterpret_cast<const f32x4*>(wr + k0 + 16 * u + 4 * g);
            }
        } else {
#pragma unroll
            for (int u = 0; u < STEPS; ++u) {
                a[u] = load_cols4(xr, k0 + 16 * u + 4 * g, k_end, x_vec != 0);
                b[u] = load_cols4(wr, k0 + 16 * u + 4 * g, k_end, w_vec != 0);
            }
        }
#pragma unroll
        for (int u = 0; u < STEPS; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][j], b[u][j], acc, 0, 0, 0);
    }
    red[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    const f32x4 sum = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    // lane holds samples m0 + 4 g + i, hidden unit n0 + r
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (m0 + 4 * g + i < B) part[((int64_t)(m0 + 4 * g + i) * gridDim.z + blockIdx.z) * hid + n0 + r] = sum[i];
}

void launch_mlp_fc1(hipStream_t s, const float* x, const BatchRows& rows, const float* W, int B, int hid, int K, float* part, bool rides) {
    const int x_vec = K % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0, w_vec = K % 4 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0;
    const dim3 grid((B + 15) / 16, hid / 16, mlp_splits(K, rides));
    const int k_wave = rides ? MLP_PART / 4 : ((K + 4 * MLP_SPLITS - 1) / (4 * MLP_SPLITS) + 15) / 16 * 16;
    if (rides) hipLaunchKernelGGL(mlp_fc1_kernel<4>, grid, dim3(256), 0, s, x, rows, W, B, hid, K, k_wave, part, x_vec, w_vec);
    else hipLaunchKernelGGL(mlp_fc1_kernel<6>, grid, dim3(256), 0, s, x, rows, W, B, hid, K, k_wave, part, x_vec, w_vec);
}

__device__ __forceinline__ void sgd_one(float& p, float& m, float grad, const bls_sgd& o) {
    const float buf = __fmaf_rn(o.momentum, m, __fmaf_rn(o.weight_decay, p, grad));
    m = buf;
    p = __fmaf_rn(-o.lr, buf, p);
}

// Four weights of a row that starts at `at`, from input n, and their momentum; zeros past the end
__device__ __forceinline__ void mlp_load_weights(f32x4& pv, f32x4& mv, const float* params, const float* momentum, int64_t at, int n, int K, int p_vec) {
    pv = mv = f32x4{0.f, 0.f, 0.f, 0.f};
    if (n < K) {
        pv = load_cols4(params + at, n, K, p_vec != 0);
        mv = load_cols4(momentum + at, n, K, p_vec != 0);
    }
}

// Gradients and update of every parameter, by workgroups of three kinds in one launch:
//   the second layer: 64 weights of one class (and, from the first 64, its bias), four slices of the batch folded through LDS;
//   the first layer's bias: 64 hidden units, likewise;
//   the first layer's weights: 16 hidden units x 256 inputs, a wave 16 x 64: lane l supplies hidden unit l % 16 and inputs
//   4 (l % 16) .. + 3 of samples 4 (l / 16) + j, one 16-byte load of x for four products, and owns four rows of four neighbouring
//   weights, which it updates with 16-byte accesses.  Two steps (32 samples) of loads are in flight together.
// The small kinds come first: they are the longer chains.
// NEXT: a workgroup of the last kind then has 16 x 256 weights of the next step and computes that step's partial sums
// part[b][z][h] over its 256 inputs (z = their block): the weights pass through LDS into the layout of a factor, the rows of
// the next batch are requested before anything else.  Sums as in mlp_fc1_kernel: a chain per quarter of the
// part, added in pairs, so that the bits do not depend on which of the two a step's sums come from.
// AHEAD: weights and momentum are requested before the sums, and the loads of 32 samples before the products of the 32 before them.
// Not for large batches and narrow layers: of the former several workgroups share a compute unit, and their number hides more than
// the registers of those requests (8 steps of 200 samples with 1024 hidden units 621 us, 636 with them; 512 units and 256 samples
// 434 / 439), the latter gain nothing (128 units and 200 samples 229.5 / 229.9).
template <bool NEXT, bool AHEAD>
__global__ __launch_bounds__(256) void mlp_update_kernel(float* __restrict__ params, float* __restrict__ momentum, MlpOffsets off,
                                                         const float* __restrict__ x, BatchRows rows, const float* __restrict__ h,
                                                         const float* __restrict__ dlogits, const float* __restrict__ dpre, int B, int hid, int C,
                                                         int K, bls_sgd opt, int x_vec, int p_vec, BatchRows next, float* __restrict__ part) {
    __shared__ float red[4][64];
    __shared__ int64_t at[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int f_blocks = (hid + 63) / 64;
    int blk = blockIdx.x;
    if (blk < (C + 1) * f_blocks) {
        const int c = blk / f_blocks, f = (blk - c * f_blocks) * 64 + lane;
        float acc = 0.f;
        if (c < C) {
            if (f < hid) {
#pragma unroll 8
                for (int b = wave; b < B; b += 4) acc = __fmaf_rn(dlogits[(int64_t)b * C + c], h[(int64_t)b * hid + f], acc);
            }
        } else if (f < hid) {
#pragma unroll 8
            for (int b = wave; b < B; b += 4) acc += dpre[(int64_t)b * hid + f];
        }
        red[wave][lane] = acc;
        __syncthreads();
        if (wave == 0 && f < hid) {
            const int64_t o = c < C ? off.fc2_w + (int64_t)c * hid + f : off.fc1_b + f;
            sgd_one(params[o], momentum[o], (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]), opt);
        }
        if (c < C && blk == c * f_blocks && wave == 1) {
            float sum = 0.f;
            for (int b = lane; b < B; b += 64) sum += dlogits[(int64_t)b * C + c];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
            if (lane == 0) sgd_one(params[off.fc2_b + c], momentum[off.fc2_b + c], sum, opt);
        }
        return;
    }
    blk -= (C + 1) * f_blocks;
    const int r = lane & 15, g = lane >> 4;
    const int n_blocks = (K + MLP_PART - 1) / MLP_PART;
    const int m0 = (blk / n_blocks) * 16, z = blk % n_blocks, n = z * 256 + wave * 64 + 4 * r;
    // the wave's first 16 samples of the next batch: lane l supplies row l % 16 and, in a step of 16 inputs, four from 4 (l / 16)
    f32x4 xn[NEXT ? 16 : 1];
    auto load_next = [&](int b0) {
        const float* row = x + pool_row(next, min(b0 + r, B - 1)) * K;   // rows past the batch repeat its last one and are not stored
        if (x_vec && z * 256 + 256 <= K) {   // uniform, so that all sixteen are in flight together
#pragma unroll
            for (int u = 0; u < (NEXT ? 16 : 0); ++u) xn[u] = *reinterpret_cast<const f32x4*>(row + z * 256 + 16 * u + 4 * g);
        } else {
#pragma unroll
            for (int u = 0; u < (NEXT ? 16 : 0); ++u) xn[u] = load_cols4(row, z * 256 + 16 * u + 4 * g, K, x_vec != 0);
        }
    };
    if (NEXT && 16 * wave < B) load_next(16 * wave);
    const int nn = n < K ? n : 0;   // a lane past the last input reads the first ones and stores nothing
    f32x4 pv[4], mv[4];
    if constexpr (AHEAD) {
#pragma unroll
        for (int i = 0; i < 4; ++i) mlp_load_weights(pv[i], mv[i], params, momentum, off.fc1_w + (int64_t)(m0 + 4 * g + i) * K, n, K, p_vec);
    }
    f32x4 acc[4] = {};
    for (int b0 = 0; b0 < B; b0 += 256) {
        __syncthreads();
        at[tid] = pool_row(rows, min(b0 + tid, B - 1));
        __syncthreads();
        const int b_end = min(B, b0 + 256);
        float a[AHEAD ? 2 : 1][8];
        f32x4 v[AHEAD ? 2 : 1][8];
        auto fetch = [&](int k0, float (&a)[8], f32x4 (&v)[8]) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int b = min(k0 + 16 * (j >> 2) + 4 * g + (j & 3), b_end - 1);
                a[j] = dpre[(int64_t)b * hid + m0 + r];
                const float* row = x + at[b - b0] * K;
                if (x_vec) v[j] = *reinterpret_cast<const f32x4*>(row + nn);
                else v[j] = load_cols4(row, nn, K, false);
            }
        };
        auto multiply = [&](int k0, const float (&a)[8], const f32x4 (&v)[8]) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool ok = k0 + 16 * (j >> 2) + 4 * g + (j & 3) < b_end;   // samples past the batch: zero factors
                const float aj = ok ? a[j] : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(aj, ok ? v[j][q] : 0.f, acc[q], 0, 0, 0);
            }
        };
        if constexpr (AHEAD) {
            fetch(b0, a[0], v[0]);
            for (int k0 = b0; k0 < b_end; k0 += 64) {
                if (k0 + 32 < b_end) fetch(k0 + 32, a[1], v[1]);
                multiply(k0, a[0], v[0]);
                if (k0 + 32 >= b_end) break;
                if (k0 + 64 < b_end) fetch(k0 + 64, a[0], v[0]);
                multiply(k0 + 32, a[1], v[1]);
            }
        } else {
            for (int k0 = b0; k0 < b_end; k0 += 32) {
                fetch(k0, a[0], v[0]);
                multiply(k0, a[0], v[0]);
            }
        }
    }
    if constexpr (!AHEAD) {
#pragma unroll
        for (int i = 0; i < 4; ++i) mlp_load_weights(pv[i], mv[i], params, momentum, off.fc1_w + (int64_t)(m0 + 4 * g + i) * K, n, K, p_vec);
    }
    // lane holds hidden units m0 + 4 g + i, inputs n .. n + 3
    constexpr int PITCH = 256 + 4;
    __shared__ __attribute__((aligned(16))) float w_lds[NEXT ? 16 * PITCH : 4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float* p = params + off.fc1_w + (int64_t)(m0 + 4 * g + i) * K + n;
        float* m = momentum + off.fc1_w + (int64_t)(m0 + 4 * g + i) * K + n;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float ps = pv[i][q], ms = mv[i][q];
            sgd_one(ps, ms, n + q < K ? acc[q][i] : 0.f, opt);
            pv[i][q] = n + q < K ? ps : 0.f;
            mv[i][q] = ms;
        }
        if (p_vec && n < K) {
            *reinterpret_cast<f32x4*>(p) = pv[i];
            *reinterpret_cast<f32x4*>(m) = mv[i];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (n + q < K) {
                    p[q] = pv[i][q];
                    m[q] = mv[i][q];
                }
        }
        if (NEXT) *reinterpret_cast<f32x4*>(w_lds + (4 * g + i) * PITCH + wave * 64 + 4 * r) = pv[i];
    }
    if constexpr (NEXT) {
        __syncthreads();
        for (int b0 = 16 * wave; b0 < B; b0 += 64) {
            f32x4 sum[4] = {};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                f32x4 w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const f32x4*>(w_lds + r * PITCH + 64 * q + 16 * u + 4 * g);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) sum[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(xn[4 * q + u][j], w[q][j], sum[q], 0, 0, 0);
            }
            const f32x4 v = (sum[0] + sum[1]) + (sum[2] + sum[3]);
            if (b0 + 64 < B) load_next(b0 + 64);
            // lane holds samples b0 + 4 g + i, hidden unit m0 + r
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (b0 + 4 * g + i < B) part[((int64_t)(b0 + 4 * g + i) * n_blocks + z) * hid + m0 + r] = v[i];
        }
    }
}

void launch_mlp_update(hipStream_t s, float* params, float* momentum, const MlpOffsets& off, const float* x, const BatchRows& rows, const float* h,
                       const float* dlogits, const float* dpre, int B, int hid, int C, int K, const bls_sgd& opt, bool rides, const BatchRows* next, float* part) {
    const int x_vec = K % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
    const int p_vec = K % 4 == 0 && (reinterpret_cast<uintptr_t>(params + off.fc1_w) | reinterpret_cast<uintptr_t>(momentum + off.fc1_w)) % 16 == 0;
    const unsigned blocks = (unsigned)((C + 1) * ((hid + 63) / 64) + (hid / 16) * ((K + 255) / 256));
#define MLP_UPDATE(NEXT, AHEAD) \
    hipLaunchKernelGGL((mlp_update_kernel<NEXT, AHEAD>), dim3(blocks), dim3(256), 0, s, params, momentum, off, x, rows, h, dlogits, dpre, B, hid, C, K, opt, x_vec, \
                       p_vec, next ? *next : BatchRows{}, part)
    if (next) MLP_UPDATE(true, true);
    else if (rides) MLP_UPDATE(false, true);
    else MLP_UPDATE(false, false);
#undef MLP_UPDATE
}
