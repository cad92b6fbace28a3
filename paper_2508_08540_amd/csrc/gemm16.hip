// GEMM on the bf16 matrix cores with both operands stored in bf16:
//   C[m][n] = alpha * sum_k A(m,k) B(n,k) [+ bias[n]] [+ R[m][n]],  fp32 sums.
// A(m,k) is A[m*lda + k] or, with a_kmajor, A[k*lda + m]; likewise B(n,k); or either in panels of 32 columns (Gemm16Desc); batch index z = z1 * inner + z2 as in the
// fp32 products.  The result goes out as fp32 (C), as bf16 rounded to nearest even (C16), as bf16 gelu(C) (G16), or any
// combination; bias and R are fp32.  With splits > 1 the K range is cut into fp32 partials that launch_split_reduce adds in
// split order.  The B tile is the first operand of v_mfma_f32_16x16x32_bf16, so that lane (r, g) holds C[m = r][n = 4g .. 4g+3] of
// a 16 x 16 block: four adjacent outputs.
//
// Two kernels.  gemm16_direct_kernel takes every product whose rows start on 16-byte boundaries: its tiles go from global
// memory straight into LDS.  gemm16_kernel takes the others (odd widths), element by element where it has to: 128 x 128 tile of
// C per workgroup, four waves as 2 x 2, each 64 x 64 = 4 x 4 blocks.  K advances 32 at a time through two LDS buffers [128 rows][32 k]
// with a row pitch of 96 bytes (measured: the 16-byte operand reads, 16 rows x 4 k groups per instruction, run at the full LDS
// rate when the pitch is 32 bytes more than a multiple of 64, at half of it with an odd number of 16-byte units such as 80 or 144
// bytes); the next two steps' global loads are in flight in registers while the matrix instructions run.
#include <type_traits>

#include "act.h"
#include "kernels.h"

#define G16_TILE 128
#define G16_K 32
#define G16_PITCH 48   // bf16 elements per LDS row (96 bytes)
#define G16_RUN 8      // steps in a running sum of a weight gradient

typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_v __attribute__((ext_vector_type(8)));
typedef float f32x2_v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_v){lo, hi}, bf16x2_v));
}

// ---- operands through registers (gemm16_kernel) ---------------------------------------------------------------------------
// Two 16-byte pieces per thread for the 128 rows of an operand tile.
// Row-major operand: piece `sub` covers, with f = tid + 256 sub, row f >> 2, k = 8 (f & 3) .. + 7.
// K-major operand: the thread takes k = 2 kp + sub for the eight rows of chunk c, kp = (tid >> 2) & 15,
// c = 4 (tid >> 6) + (tid & 3); the two pieces are interleaved into (k, k+1) pairs on the way into LDS.
template <bool KMAJOR>
__device__ __forceinline__ void g16_piece(int sub, int& row, int& k) {
    if (KMAJOR) {
        row = 8 * (4 * (int)(threadIdx.x >> 6) + (int)(threadIdx.x & 3));
        k = 2 * (int)((threadIdx.x >> 2) & 15) + sub;
    } else {
        const int f = threadIdx.x + 256 * sub;
        row = f >> 2;
        k = 8 * (f & 3);
    }
}

// Checked fetch: any shape and alignment, element by element where a 16-byte load is not possible.
template <bool KMAJOR>
__device__ __forceinline__ void g16_fetch(const bf16_t* __restrict__ P, int ld, int rows, int row0, int k0, int k_end, bool vec, u32x4 (&v)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int row, k;
        g16_piece<KMAJOR>(i, row, k);
        row += row0;
        k += k0;
        u32x4 w = {0u, 0u, 0u, 0u};
        if (KMAJOR) {
            if (k < k_end) {
                const bf16_t* p = P + (int64_t)k * ld + row;
                if (vec && row + 7 < rows) {
                    w = *reinterpret_cast<const u32x4*>(p);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (row + j < rows) w[j >> 1] |= (uint32_t)p[j] << (16 * (j & 1));
                }
            }
        } else {
            if (row < rows) {
                const bf16_t* p = P + (int64_t)row * ld + k;
                if (vec && k + 7 < k_end) {
                    w = *reinterpret_cast<const u32x4*>(p);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (k + j < k_end) w[j >> 1] |= (uint32_t)p[j] << (16 * (j & 1));
                }
            }
        }
        v[i] = w;
    }
}

template <bool KMAJOR>
__device__ __forceinline__ void g16_put(bf16_t* __restrict__ S, const u32x4 (&v)[2]) {
    int row, k;
    if (KMAJOR) {
        g16_piece<true>(0, row, k);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // rows row + 2j and row + 2j + 1: the low and the high halves of word j of both pieces
            *reinterpret_cast<uint32_t*>(S + (row + 2 * j) * G16_PITCH + k) = __builtin_amdgcn_perm(v[1][j], v[0][j], 0x05040100u);
            *reinterpret_cast<uint32_t*>(S + (row + 2 * j + 1) * G16_PITCH + k) = __builtin_amdgcn_perm(v[1][j], v[0][j], 0x07060302u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            g16_piece<false>(i, row, k);
            *reinterpret_cast<u32x4*>(S + row * G16_PITCH + k) = v[i];
        }
    }
}

// GELU (erf form) of the bf16 mode's epilogues, x Phi(x), without the branches of erff.  Two forms of Phi meet at |x| = 1.5:
//   inside, 1/2 + x q(x^2), whose product is formed before the half is added, so that half a unit of x q and the rounding of the sum
//   are all its error; q is a constant less x^2 times a polynomial, least squares reweighted to the largest error (6e-9 of Phi);
//   outside, Phi(-|x|) = exp(-x^2 / 2) t P(t), t = 1 / (1 + 0.4 |x|), P fitted to the Mills ratio in the same way (6e-8).
// Relative rms error of x Phi(x) on the device in units of 1e-8, on [-4, -1.5], [-1.5, -1/2], [-1/2, 0], [0, 1/2], [1/2, 1.5], [1.5, 4]:
// 20, 9.5, 3.7, 4.0, 3.7, 2.9 (with erff 6000, 11.9, 3.8, 4.0, 3.9, 3.3; the outer form alone, 2 % faster over four steps of the
// 6-layer encoder, has 11.9 and 9.2 around 0).
#define GELU_LOG2E_2 -0.7213475204444817f   // exp(-x^2 / 2) = 2^(x^2 times this)
__device__ __forceinline__ float gelu_phi(float x, float s, float e) {   // s = x^2, e = exp(-s / 2)
    const float ax = fabsf(x), t = __builtin_amdgcn_rcpf(__fmaf_rn(0.4f, ax, 1.f));
    float p = 0.06783060729503632f;
    p = __fmaf_rn(p, t, -0.18599045276641846f);
    p = __fmaf_rn(p, t, 0.10517537593841553f);
    p = __fmaf_rn(p, t, 0.0555267333984375f);
    p = __fmaf_rn(p, t, 0.13903170824050903f);
    p = __fmaf_rn(p, t, 0.15909291803836823f);
    p = __fmaf_rn(p, t, 0.1595963090658188f);
    const float tail = p * t * e;
    float q = -3.950671896291169e-7f;
    q = __fmaf_rn(q, s, 8.600311957707163e-6f);
    q = __fmaf_rn(q, s, -1.140362728619948e-4f);
    q = __fmaf_rn(q, s, 1.1860835365951061e-3f);
    q = __fmaf_rn(q, s, -9.973009116947651e-3f);
    q = __fmaf_rn(q, s, 6.64902925491333e-2f);
    q = __fmaf_rn(q, s, 1.1335170e-8f);   // what the next constant exceeds 1 / sqrt(2 pi) by
    const float near = 0.5f + __fmaf_rn(x, 0.3989422917366028f, -(x * q));
    return ax < 1.5f ? near : x < 0.f ? tail : 1.f - tail;
}
__device__ __forceinline__ float gelu_for_bf16(float x) {
    const float s = x * x;
    return x * gelu_phi(x, s, __builtin_amdgcn_exp2f(s * GELU_LOG2E_2));
}
// its derivative Phi(x) + x phi(x); rms error on the same intervals: 0.6, 1.5, 1.4, 2.5, 4.0, 3.9 (with erff and expf 1.1, 1.7, 1.4,
// 2.6, 4.0, 4.2).
__device__ __forceinline__ float gelu_df_for_bf16(float x) {
    const float s = x * x, e = __builtin_amdgcn_exp2f(s * GELU_LOG2E_2);
    return __fmaf_rn(x * 0.3989422804014327f, e, gelu_phi(x, s, e));
}

__device__ __forceinline__ void g16_tile_of_block(int& tile_x, int& tile_y) {
    // launch slot -> tile such that each of the eight XCDs (round-robin over launch slots) walks a contiguous tile range
    const int nx = gridDim.x, tiles = nx * gridDim.y;
    int id = blockIdx.y * nx + blockIdx.x;
    if ((tiles & 7) == 0) id = (id & 7) * (tiles >> 3) + (id >> 3);
    tile_y = id / nx;
    tile_x = id - tile_y * nx;
}

// element (m, n) of the bf16 outputs: panels of 32 columns c16_panel apart (row-major: 32 apart)
__device__ __forceinline__ int64_t g16_at16(const Gemm16Desc& d, int m, int n) { return (n >> 5) * d.c16_panel + (int64_t)m * d.ldc16 + (n & 31); }

// Stores a wave's 64 x 64 block; lane (r, g) holds acc[mt][nt][i] = C[m_base + 16 mt + r][n_base + 16 nt + 4 g + i].
template <bool VEC, bool GELU>
__device__ __forceinline__ void g16_store_block(const Gemm16Desc& d, const f32x4 (&acc)[4][4], int m_base, int n_base, float* C, bf16_t* C16,
                                                bf16_t* G16, const float* R, const float* bias, int ldc, bool plain, int r, int g) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        const int m = m_base + 16 * mt + r;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int n = n_base + 16 * nt + 4 * g;
            if (VEC) {
                // the block lies inside C and rows allow 16-byte accesses
                f32x4 v = acc[mt][nt];
                const int64_t at = (int64_t)m * ldc + n;
                if (!plain) {
                    v *= d.alpha;
                    if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
                    if (R) v += *reinterpret_cast<const f32x4*>(R + at);
                }
                if (C) *reinterpret_cast<f32x4*>(C + at) = v;
                if (C16) *reinterpret_cast<u32x2*>(C16 + g16_at16(d, m, n)) = u32x2{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
                if (GELU && G16) {
                    f32x4 q;
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = gelu_for_bf16(v[i]);
                    *reinterpret_cast<u32x2*>(G16 + g16_at16(d, m, n)) = u32x2{pack2_bf16(q[0], q[1]), pack2_bf16(q[2], q[3])};
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (m < d.M && n + i < d.N) {
                        float v = acc[mt][nt][i];
                        const int64_t at = (int64_t)m * ldc + n + i;
                        if (!plain) {
                            v *= d.alpha;
                            if (bias) v += bias[n + i];
                            if (R) v += R[at];
                        }
                        if (C) C[at] = v;
                        if (C16) C16[g16_at16(d, m, n + i)] = (bf16_t)(pack2_bf16(v, 0.f) & 0xffffu);
                        if (GELU && G16) G16[g16_at16(d, m, n + i)] = (bf16_t)(pack2_bf16(gelu_for_bf16(v), 0.f) & 0xffffu);
                    }
                }
            }
        }
    }
}

// Softmax statistics of a wave's 64 columns for each of its 64 rows: ce_part[2 * tile_x + wn][m] = (max, sum of
// exp(v - max)) over the columns that exist, and the value in column ce_targets[m] goes to ce_tlogit[m] when this wave
// holds it.  A later pass folds the pairs of a row in index order.  The product is taken without bias.
__device__ __forceinline__ void g16_ce_block(const Gemm16Desc& d, const f32x4 (&acc)[4][4], int m_base, int n_base, int part_idx, int r, int g) {
    const bool full = n_base + 64 <= d.N;   // uniform: every column of the block exists
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        const int m = m_base + 16 * mt + r;
        const int tgt = m < d.M ? d.ce_targets[m] : -1;
        const int t_local = tgt - n_base - 4 * g;   // column of the target among this lane's 16, as 16 nt + i
        float v[16];
        float mx = -INFINITY, at_target = 0.f;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float q = acc[mt][nt][i] * d.alpha;
                if (!full && n_base + 16 * nt + 4 * g + i >= d.N) q = -INFINITY;
                v[4 * nt + i] = q;
                mx = fmaxf(mx, q);
                at_target = t_local == 16 * nt + i ? q : at_target;
            }
        if (t_local >= 0 && t_local < 64 && (t_local & 12) == 0) d.ce_tlogit[m] = at_target;
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        float sum = 0.f;
        if (mx > -INFINITY)
#pragma unroll
            for (int j = 0; j < 16; ++j) sum += __expf(v[j] - mx);   // hardware exponential: 64 per lane, the accurate one would double the tile time
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        if (g == 0 && m < d.M) *reinterpret_cast<f32x2_v*>(d.ce_part + 2 * ((int64_t)part_idx * d.M + m)) = f32x2_v{mx, sum};
    }
}

// EPI: 0 plain epilogue, 1 also writes gelu(C) (its code stays out of the other instantiations), 2 softmax statistics
template <bool AK, bool BK, int EPI>
__global__ __launch_bounds__(256, AK ? 2 : 3) void gemm16_kernel(Gemm16Desc d) {
    __shared__ __attribute__((aligned(16))) bf16_t As[2][G16_TILE * G16_PITCH], Bs[2][G16_TILE * G16_PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    int tile_x, tile_y;
    g16_tile_of_block(tile_x, tile_y);
    const int m0 = tile_y * G16_TILE, n0 = tile_x * G16_TILE;
    const int split = blockIdx.z % d.splits, z = blockIdx.z / d.splits;
    const int z1 = z / d.inner, z2 = z - z1 * d.inner;
    const bf16_t* A = d.A + z1 * d.sa1 + z2 * d.sa2;
    const bf16_t* B = d.B + z1 * d.sb1 + z2 * d.sb2;
    const int k_begin = split * d.k_chunk;
    const int k_end = min(d.K, k_begin + d.k_chunk);
    const bool avec = d.a_vec != 0, bvec = d.b_vec != 0;

    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sum[AK ? 4 : 1][AK ? 4 : 1] = {};   // weight gradients: of the runs that are over
    int in_run = 0;

    // each tile row of C starts its walk over K at a different step and wraps around, so that workgroups in flight
    // read different k ranges (rows with a power-of-two pitch otherwise meet in few memory channels)
    const int steps = (k_end - k_begin + G16_K - 1) / G16_K;
    const int rot = steps > 0 ? tile_y % steps : 0;
    auto k_of = [&](int i) {
        const int sidx = i + rot < steps ? i + rot : i + rot - steps;
        return k_begin + sidx * G16_K;
    };
    // Two K steps of global loads are in flight (register sets 0 and 1, used in turn) while a third is multiplied
    // out of LDS: with one to three workgroups per compute unit it is the bytes in flight that bound the rate.
    u32x4 pa0[2], pb0[2], pa1[2], pb1[2];
    auto fetch = [&](int k, u32x4 (&pa)[2], u32x4 (&pb)[2]) {
        g16_fetch<AK>(A, d.lda, d.M, m0, k, k_end, avec, pa);
        g16_fetch<BK>(B, d.ldb, d.N, n0, k, k_end, bvec, pb);
    };
    auto compute = [&](int buf) {
        const bf16_t* as = As[buf] + (wm * 64 + r) * G16_PITCH + 8 * g;
        const bf16_t* bs = Bs[buf] + (wn * 64 + r) * G16_PITCH + 8 * g;
        bf16x8_v a[4], b[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = *reinterpret_cast<const bf16x8_v*>(as + 16 * t * G16_PITCH);
#pragma unroll
        for (int t = 0; t < 4; ++t) b[t] = *reinterpret_cast<const bf16x8_v*>(bs + 16 * t * G16_PITCH);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[nt], a[mt], acc[mt][nt], 0, 0, 0);
        if constexpr (AK)
            if (++in_run == G16_RUN) {
                in_run = 0;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt) {
                        sum[mt][nt] += acc[mt][nt];
                        acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
    };
    if (steps > 0) {
        fetch(k_of(0), pa0, pb0);
        g16_put<AK>(As[0], pa0);
        g16_put<BK>(Bs[0], pb0);
    }
    if (steps > 1) fetch(k_of(1), pa0, pb0);
    __syncthreads();
    int i = 0;
    // steady state, two steps per turn: every fetch and store is unconditional here, so that the wait before a store
    // into LDS counts the younger set's loads as still in flight
    for (; i + 3 < steps; i += 2) {
        fetch(k_of(i + 2), pa1, pb1);
        compute(0);
        g16_put<AK>(As[1], pa0);
        g16_put<BK>(Bs[1], pb0);
        __syncthreads();
        fetch(k_of(i + 3), pa0, pb0);
        compute(1);
        g16_put<AK>(As[0], pa1);
        g16_put<BK>(Bs[0], pb1);
        __syncthreads();
    }
    // the last (up to three) steps
    while (i < steps) {
        // LDS buffer 0 holds step i, register set 0 step i + 1
        if (i + 2 < steps) fetch(k_of(i + 2), pa1, pb1);
        compute(0);
        if (i + 1 < steps) {
            g16_put<AK>(As[1], pa0);
            g16_put<BK>(Bs[1], pb0);
        }
        __syncthreads();
        if (++i >= steps) break;
        // LDS buffer 1 holds step i, register set 1 step i + 1
        if (i + 2 < steps) fetch(k_of(i + 2), pa0, pb0);
        compute(1);
        if (i + 1 < steps) {
            g16_put<AK>(As[0], pa1);
            g16_put<BK>(Bs[0], pb1);
        }
        __syncthreads();
        ++i;
    }
    if constexpr (AK)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) acc[mt][nt] += sum[mt][nt];

    const bool plain = d.splits > 1;   // partial sums go out as they are; the reduction applies the epilogue
    const int64_t zoff = z1 * d.sc1 + z2 * d.sc2;
    float* C = plain ? d.part + ((int64_t)z * d.splits + split) * d.part_stride : d.C ? d.C + zoff : nullptr;
    const int64_t zoff16 = z1 * d.sc1_16 + z2 * d.sc2_16;
    bf16_t* C16 = (plain || !d.C16) ? nullptr : d.C16 + zoff16;
    bf16_t* G16 = (plain || !d.G16) ? nullptr : d.G16 + zoff16;
    const float* R = (plain || !d.R) ? nullptr : d.R + zoff;
    const float* bias = (plain || !d.bias) ? nullptr : d.bias + z1 * d.sbias1;
    const int ldc = plain ? d.N : d.ldc;
    const int m_base = m0 + wm * 64, n_base = n0 + wn * 64;
    if (EPI == 2) g16_ce_block(d, acc, m_base, n_base, 2 * tile_x + wn, r, g);   // its own instantiation: the statistics cost registers
    const bool vec = (plain ? (d.N & 3) == 0 : d.c_vec != 0) && m_base + 64 <= d.M && n_base + 64 <= d.N;
    if (vec) g16_store_block<true, EPI == 1>(d, acc, m_base, n_base, C, C16, G16, R, bias, ldc, plain, r, g);
    else g16_store_block<false, EPI == 1>(d, acc, m_base, n_base, C, C16, G16, R, bias, ldc, plain, r, g);
}

// ---- tiles straight into LDS (gemm16_direct_kernel) --------------------------------------------------------------------------
//
// Workgroup = 32 WMB x 32 WNB tile of C, four waves as 2 x 2, each 16 WMB x 16 WNB.  K advances 32 KS at a time through
// GD16_STAGES LDS buffers [row][32 k] that global_load_lds fills (16 bytes per lane, 1 KB of consecutive LDS per
// instruction): no staging registers, no LDS store instructions, two steps of loads in flight.  One barrier per step: a wave
// waits for its own loads of the step (counted, the younger step stays in flight), the barrier makes everybody's visible and
// frees the buffer read a step ago.  Rows are 64 bytes; piece c (16 bytes) of a row sits at place c ^ gd16_place(row),
// so that the 16-byte operand reads, 16 rows x 4 pieces, are free of bank conflicts.  Rows past the end are clamped to the last one (they only
// feed outputs that are never stored), pieces past the end of K are zeroed in LDS in the last step.
#define GD16_STAGES 3   // the last two steps' waits count on it
typedef __attribute__((address_space(1))) const void gd16_global_ptr;
typedef __attribute__((address_space(3))) void gd16_lds_ptr;

// A 16-byte LDS read of a wave proceeds 16 lanes at a time, but not 16 consecutive ones: eight rows of one piece together with
// eight other rows of its neighbour.  With this permutation (0, 2, 3, 1 over the row quads) those fall on different banks.
__device__ __forceinline__ int gd16_place(int quad) { return (((quad ^ (quad >> 1)) & 1) << 1) | ((quad >> 1) & 1); }

// Epilogue.  Rows of a row-major B are dealt to the matrix blocks so that blocks 2p and 2p + 1 of a lane hold eight neighbouring columns
// n_base + 32 p + 8 g ..: 16-byte stores of bf16, 32 bytes of fp32.  Everything the epilogue reads is requested before the
// first store of a group of block rows (the compiler has to assume that a store changes what a later load reads, so a
// load behind a store is a memory round trip of its own: 32 of them per tile cost more than the matrix loop of K = 512).
template <bool PAIRED>
__device__ __forceinline__ int gd16_column(int nt, int g) { return PAIRED ? 32 * (nt >> 1) + 8 * g + 4 * (nt & 1) : 16 * nt + 4 * g; }

template <bool PAIRED, int WMB, int WNB, bool GELU>
__device__ __forceinline__ void gd16_store(const Gemm16Desc& d, float alpha, f32x4 (&acc)[WMB][WNB], int m_base, int n_base, float* C, bf16_t* C16, bf16_t* G16,
                                           const float* R, const float* bias, int ldc, bool plain, int r, int g) {
    if (!plain) {
        if (alpha != 1.f)
#pragma unroll
            for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt) acc[mt][nt] *= alpha;
        if (bias) {
            f32x4 b[WNB];
#pragma unroll
            for (int nt = 0; nt < WNB; ++nt) b[nt] = *reinterpret_cast<const f32x4*>(bias + n_base + gd16_column<PAIRED>(nt, g));
#pragma unroll
            for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt) acc[mt][nt] += b[nt];
        }
    }
    constexpr int GR = WMB >= 8 ? 4 : 2;   // block rows per group: what the registers beside the accumulators hold
#pragma unroll
    for (int m4 = 0; m4 < WMB; m4 += GR) {
        if (!plain && R) {
            f32x4 rv[GR][WNB];
#pragma unroll
            for (int k = 0; k < GR; ++k)
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt)
                    rv[k][nt] = *reinterpret_cast<const f32x4*>(R + (int64_t)(m_base + 16 * (m4 + k) + r) * ldc + n_base + gd16_column<PAIRED>(nt, g));
#pragma unroll
            for (int k = 0; k < GR; ++k)
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt) acc[m4 + k][nt] += rv[k][nt];
        }
#pragma unroll
        for (int k = 0; k < GR; ++k) {
            const int64_t at = (int64_t)(m_base + 16 * (m4 + k) + r) * ldc + n_base;
#pragma unroll
            for (int p = 0; p < WNB / 2; ++p) {
                const f32x4 v0 = acc[m4 + k][2 * p], v1 = acc[m4 + k][2 * p + 1];
                const int64_t at0 = at + gd16_column<PAIRED>(2 * p, g), at1 = at + gd16_column<PAIRED>(2 * p + 1, g);
                if (C) {
                    *reinterpret_cast<f32x4*>(C + at0) = v0;
                    *reinterpret_cast<f32x4*>(C + at1) = v1;
                }
                const int64_t at16 = g16_at16(d, m_base + 16 * (m4 + k) + r, n_base + 32 * p) + (PAIRED ? 8 * g : 4 * g);
                auto store16 = [&](bf16_t* dst, const f32x4& q0, const f32x4& q1) {
                    const u32x4 w = {pack2_bf16(q0[0], q0[1]), pack2_bf16(q0[2], q0[3]), pack2_bf16(q1[0], q1[1]), pack2_bf16(q1[2], q1[3])};
                    if (PAIRED) {
                        *reinterpret_cast<u32x4*>(dst + at16) = w;
                    } else {
                        *reinterpret_cast<u32x2*>(dst + at16) = u32x2{w[0], w[1]};
                        *reinterpret_cast<u32x2*>(dst + at16 + 16) = u32x2{w[2], w[3]};
                    }
                };
                if (C16) store16(C16, v0, v1);
                if (GELU && G16) {
                    f32x4 q0, q1;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        q0[i] = gelu_for_bf16(v0[i]);
                        q1[i] = gelu_for_bf16(v1[i]);
                    }
                    store16(G16, q0, q1);
                }
            }
        }
    }
}

// The same for tiles at the edge of C and for outputs without 16-byte rows
template <bool PAIRED, int WMB, int WNB, bool GELU>
__device__ __forceinline__ void gd16_store_edge(const Gemm16Desc& d, float alpha, const f32x4 (&acc)[WMB][WNB], int m_base, int n_base, float* C, bf16_t* C16,
                                                bf16_t* G16, const float* R, const float* bias, int ldc, bool plain, int r, int g) {
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m_base + 16 * mt + r;
        if (m >= d.M) continue;
#pragma unroll
        for (int nt = 0; nt < WNB; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = n_base + gd16_column<PAIRED>(nt, g) + i;
                if (n < d.N) {
                    float v = acc[mt][nt][i];
                    const int64_t at = (int64_t)m * ldc + n;
                    if (!plain) {
                        v *= alpha;
                        if (bias) v += bias[n];
                        if (R) v += R[at];
                    }
                    if (C) C[at] = v;
                    if (C16) C16[g16_at16(d, m, n)] = (bf16_t)(pack2_bf16(v, 0.f) & 0xffffu);
                    if (GELU && G16) G16[g16_at16(d, m, n)] = (bf16_t)(pack2_bf16(gelu_for_bf16(v), 0.f) & 0xffffu);
                }
            }
    }
}

// Softmax statistics of a wave's 64 columns for each of its rows, as g16_ce_block: (max, sum of exp(v - max)) and the value in
// the target's column.  The rows' targets are requested together and the reductions of all block rows run side by side;
// the column of the target is only looked for in the rare wave that holds one.  Overwrites the block: the exponentials take the
// place of the values, so that those of all rows are independent instructions (one temporary at a time, each waited for, and a mask
// per value were a third of the 7 us that the statistics of a tile take beside another's K loop; 65 536 x 32 000 x 512
// 2144 -> 1974 us, 8192 tokens 306 -> 273).
template <int WMB>
__device__ __forceinline__ void gd16_ce(const Gemm16Desc& d, f32x4 (&acc)[WMB][4], int m_base, int n_base, int part_idx, int r, int g) {
    int tgt[WMB];
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m_base + 16 * mt + r;
        tgt[mt] = m < d.M ? d.ce_targets[m] : -1;
    }
    if (n_base + 64 > d.N) {   // uniform: columns that do not exist count as -inf
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n_base + 32 * (nt >> 1) + 8 * g + 4 * (nt & 1) + i >= d.N)
#pragma unroll
                    for (int mt = 0; mt < WMB; ++mt) acc[mt][nt][i] = -INFINITY;
    }
    float mx[WMB], sum[WMB];
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        mx[mt] = -INFINITY;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[mt] = fmaxf(mx[mt], acc[mt][nt][i]);
    }
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) mx[mt] = fmaxf(mx[mt], __shfl_xor(mx[mt], 16, 64));
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) mx[mt] = fmaxf(mx[mt], __shfl_xor(mx[mt], 32, 64));
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m_base + 16 * mt + r;
        const int t = tgt[mt] - n_base;
        if (t >= 0 && t < 64 && ((t >> 3) & 3) == g) {   // this lane holds the target's column
            float at = 0.f;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) at = (t >> 5) == (nt >> 1) && (t & 7) == 4 * (nt & 1) + i ? acc[mt][nt][i] : at;
            d.ce_tlogit[m] = at;
        }
    }
    constexpr float LOG2E = 1.4426950408889634f;
    // Hardware exponential; a row whose columns are all -inf or absent keeps a sum of 0 (its maximum says so).  The maximum is
    // taken off first: scaled and taken off in one step, its rounding would be a common factor of all terms (rms error of the
    // logarithm of the sum at maxima around 7 / 30: 7e-8 / 7e-8, in one step 2e-7 / 8e-7).
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const float ref = mx[mt] > -INFINITY ? mx[mt] : 0.f;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[mt][nt][i] = __builtin_amdgcn_exp2f((acc[mt][nt][i] - ref) * LOG2E);
        sum[mt] = 0.f;
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int mt = 0; mt < WMB; ++mt) sum[mt] += acc[mt][nt][i];
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) sum[mt] += __shfl_xor(sum[mt], 16, 64);
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) sum[mt] += __shfl_xor(sum[mt], 32, 64);
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m_base + 16 * mt + r;
        if (g == 0 && m < d.M) *reinterpret_cast<f32x2_v*>(d.ce_part + 2 * ((int64_t)part_idx * d.M + m)) = f32x2_v{mx[mt], sum[mt]};
    }
}

// Gradient of the mean cross-entropy with respect to the logits the tile holds: (exp(z - max) / sum - [column is the target]) *
// scale with the row statistics of an earlier pass over the same product; columns past n_valid (the padding of the rows) are 0.
// The exponential carries the rounding of its scaled argument as a correction; arguments below -200, where it is 0, are raised to
// that, since the correction of an infinite one is no number (a NaN stays one).
template <int WMB, int WNB>
__device__ __forceinline__ void gd16_ce_grad(const Gemm16Desc& d, const f32x4 (&acc)[WMB][WNB], int m_base, int n_base, bf16_t* C16, int r, int g) {
    f32x2_v st[WMB];
    int tgt[WMB];
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = min(m_base + 16 * mt + r, d.M - 1);
        st[mt] = *reinterpret_cast<const f32x2_v*>(d.ce_rows + 2 * (int64_t)m);
        tgt[mt] = d.ce_targets[m];
    }
    constexpr float LOG2E = 1.4426950408889634f, LOG2E_LO = 1.925963033500912e-8f, LN2 = 0.6931471805599453f;
    const bool padded = n_base + 16 * WNB > d.n_valid;   // uniform
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m_base + 16 * mt + r;
        const float f = d.ce_scale / st[mt][1];
        // few waves hold a target or the rows' padding: only they look at every column (8192 x 32 000 x 512:
        // 356 -> 344 us)
        const bool holds = __any((unsigned)(tgt[mt] - n_base) < (unsigned)(16 * WNB));
        auto columns = [&](auto every) {
#pragma unroll
            for (int p = 0; p < WNB / 2; ++p) {
                const int n = n_base + 32 * p + 8 * g;
                float q[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    float t = acc[mt][2 * p + (j >> 2)][j & 3] * d.alpha - st[mt][0];
                    t = t < -200.f ? -200.f : t;
                    const float hi = t * LOG2E, lo = __fmaf_rn(t, LOG2E, -hi) + t * LOG2E_LO;
                    const float e = __builtin_amdgcn_exp2f(hi);
                    q[j] = __fmaf_rn(e, lo * LN2, e);
                    if constexpr (decltype(every)::value) {
                        q[j] = __fmaf_rn(q[j], f, n + j == tgt[mt] ? -d.ce_scale : 0.f);
                        if (n + j >= d.n_valid) q[j] = 0.f;
                    } else {
                        q[j] *= f;
                    }
                }
                // N is a multiple of 8: a lane's eight columns are all there or none of them
                if (m < d.M && n < d.N)
                    *reinterpret_cast<u32x4*>(C16 + g16_at16(d, m, n)) = u32x4{pack2_bf16(q[0], q[1]), pack2_bf16(q[2], q[3]), pack2_bf16(q[4], q[5]), pack2_bf16(q[6], q[7])};
                __builtin_amdgcn_sched_barrier(0);   // one piece's temporaries at a time
            }
        };
        if (padded || holds) columns(std::true_type{});
        else columns(std::false_type{});
    }
}

// The tile times gelu'(U), and the column sums of the result over the wave's rows: row 2 * tile_y + wm of gelu_part.
template <int WMB, int WNB>
__device__ __forceinline__ void gd16_gelu_bwd(const Gemm16Desc& d, f32x4 (&acc)[WMB][WNB], int m_base, int n_base, int part_row, int r, int g) {
    const bool inside = m_base + 16 * WMB <= d.M && n_base + 16 * WNB <= d.N;
    f32x4 sum[WNB];
#pragma unroll
    for (int nt = 0; nt < WNB; ++nt) sum[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int GR = 2;
#pragma unroll
    for (int m4 = 0; m4 < WMB; m4 += GR) {
        f32x4 u[GR][WNB];
#pragma unroll
        for (int k = 0; k < GR; ++k)
#pragma unroll
            for (int nt = 0; nt < WNB; ++nt) {
                const int m = m_base + 16 * (m4 + k) + r, n = n_base + gd16_column<false>(nt, g);
                u[k][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (inside || (m < d.M && n < d.N)) u[k][nt] = *reinterpret_cast<const f32x4*>(d.U + (int64_t)m * d.ldc + n);   // N % 4 == 0
            }
#pragma unroll
        for (int k = 0; k < GR; ++k) {
            const bool live = inside || m_base + 16 * (m4 + k) + r < d.M;
#pragma unroll
            for (int nt = 0; nt < WNB; ++nt) {
                f32x4& v = acc[m4 + k][nt];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = live ? v[i] * d.alpha * gelu_df_for_bf16(u[k][nt][i]) : 0.f;
                sum[nt] += v;
            }
        }
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1)
#pragma unroll
        for (int nt = 0; nt < WNB; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[nt][i] += __shfl_xor(sum[nt][i], o, 64);
#pragma unroll
    for (int nt = 0; nt < WNB; ++nt) {
        const int n = n_base + gd16_column<false>(nt, g);
        if (r == nt && n < d.N) *reinterpret_cast<f32x4*>(d.gelu_part + (int64_t)part_row * d.N + n) = sum[nt];
    }
}

// Slot v (16 bytes) of an operand stage of ROWS rows: which piece of the matrix belongs there (row and k relative to the tile;
// a piece is 8 k of one row, or, k-major, 8 rows of one k).
template <bool KMAJOR, bool IS_B, int ROWS>
__device__ __forceinline__ void gd16_slot(int v, int& row, int& k) {
    if (KMAJOR) {
        constexpr int PPL = ROWS / 8;   // pieces per line
        k = v / PPL;
        const int place = v % PPL, f = ROWS >= 128 ? (k & 3) | ((k >> 1) & 4) : ((k >> 1) & 1) | ((k >> 2) & 2);
        row = 8 * (2 * ((place >> 1) ^ f) + (place & 1));
    } else {
        row = v >> 2;
        k = 8 * ((v & 3) ^ gd16_place((IS_B ? row >> 3 : row >> 2) & 3));
    }
}

// Transposing reads of the NX operands of one factor (lines of ROWS_X bf16) and the NY of the other: eight values along K for each
// of a lane's rows, two reads, lines 0 .. 3 and 4 .. 7 of its group.  All reads of a step and the wait for them are ONE assembly
// statement: nothing outside it sees a register whose data has not arrived.  (The builtin is no way out: the compiler takes it for
// a possible reader of every LDS load in flight and waits for all of them.)  Outputs are written while later addresses are still to
// be read, hence the early-clobber marks.
#define GD16_TR(i, line) "ds_read_b64_tr_b16 %[l" #i "], %[a" #i "]\n\tds_read_b64_tr_b16 %[h" #i "], %[a" #i "] offset:%[" line "]\n\t"
#define GD16_TR4(i, j, k, l, line) GD16_TR(i, line) GD16_TR(j, line) GD16_TR(k, line) GD16_TR(l, line)
#define GD16_OUT2(i, j) [l##i] "=&v"(lo[i]), [h##i] "=&v"(hi[i]), [l##j] "=&v"(lo[j]), [h##j] "=&v"(hi[j])
#define GD16_AT2(i, j) [a##i] "v"(at[i]), [a##j] "v"(at[j])
#define GD16_WAIT "s_waitcnt lgkmcnt(0)"
template <int ROWS_X, int ROWS_Y, int NX, int NY>
__device__ __forceinline__ void gd16_transposed(const uint32_t (&at)[NX + NY], u32x4 (&x)[NX + NY]) {
    constexpr int LX = 8 * ROWS_X, LY = 8 * ROWS_Y;   // bytes of four lines
    u32x2 lo[NX + NY], hi[NX + NY];
    if constexpr (NX == 2 && NY == 0)
        asm volatile(GD16_TR(0, "x") GD16_TR(1, "x") GD16_WAIT : GD16_OUT2(0, 1) : GD16_AT2(0, 1), [x] "n"(LX));
    else if constexpr (NX == 4 && NY == 0)
        asm volatile(GD16_TR4(0, 1, 2, 3, "x") GD16_WAIT : GD16_OUT2(0, 1), GD16_OUT2(2, 3) : GD16_AT2(0, 1), GD16_AT2(2, 3), [x] "n"(LX));
    else if constexpr (NX == 2 && NY == 4)
        asm volatile(GD16_TR(0, "x") GD16_TR(1, "x") GD16_TR4(2, 3, 4, 5, "y") GD16_WAIT
                     : GD16_OUT2(0, 1), GD16_OUT2(2, 3), GD16_OUT2(4, 5)
                     : GD16_AT2(0, 1), GD16_AT2(2, 3), GD16_AT2(4, 5), [x] "n"(LX), [y] "n"(LY));
    else if constexpr (NX == 4 && NY == 4)
        asm volatile(GD16_TR4(0, 1, 2, 3, "x") GD16_TR4(4, 5, 6, 7, "y") GD16_WAIT
                     : GD16_OUT2(0, 1), GD16_OUT2(2, 3), GD16_OUT2(4, 5), GD16_OUT2(6, 7)
                     : GD16_AT2(0, 1), GD16_AT2(2, 3), GD16_AT2(4, 5), GD16_AT2(6, 7), [x] "n"(LX), [y] "n"(LY));
    else {
        static_assert(NX == 4 && NY == 8, "operands per wave of the tiles the launcher chooses from");
        asm volatile(GD16_TR4(0, 1, 2, 3, "x") GD16_TR4(4, 5, 6, 7, "y") GD16_TR4(8, 9, 10, 11, "y") GD16_WAIT
                     : GD16_OUT2(0, 1), GD16_OUT2(2, 3), GD16_OUT2(4, 5), GD16_OUT2(6, 7), GD16_OUT2(8, 9), GD16_OUT2(10, 11)
                     : GD16_AT2(0, 1), GD16_AT2(2, 3), GD16_AT2(4, 5), GD16_AT2(6, 7), GD16_AT2(8, 9), GD16_AT2(10, 11), [x] "n"(LX), [y] "n"(LY));
    }
#pragma unroll
    for (int t = 0; t < NX + NY; ++t) x[t] = u32x4{lo[t][0], lo[t][1], hi[t][0], hi[t][1]};
}
#undef GD16_TR
#undef GD16_TR4
#undef GD16_OUT2
#undef GD16_AT2
#undef GD16_WAIT

// Both factors k-major: a weight gradient, whose contraction runs over all tokens.  Its sums are taken in runs of G16_RUN steps, so
// that their rounding does not grow with the length of a part; the 256-row tile has no registers for that, but takes only products
// of so many tiles that they are never split.  Over 8192 tokens the gradients of a 512-wide layer are 5.3e-8 to 6.1e-8 off the
// sum in 64 bits (relative 2-norm), in one running sum per part 7.5e-8 to 1.3e-7; four steps of the 6-layer encoder: 18.2 -> 18.45 ms.
constexpr bool gd16_runs(bool a_kmajor, int wmb) { return a_kmajor && wmb < 8; }
// waves per SIMD the registers have to allow, for 16 x 16 blocks per wave.  Of the 256 x 128 tiles those with the softmax statistics and
// with the GELU derivative do not fit the 256 of two waves: 25 and 22 registers go to memory and back once in their epilogues,
// none in the K loop (about 100 bytes a lane and tile, against 512 of results and 1 to 2 KB of operands).
constexpr int gd16_waves(bool runs, int blocks) { return blocks >= (runs ? 16 : 32) ? 2 : 3; }

template <bool AK, bool BK, int EPI, int WMB, int WNB, int KS>
__global__ __launch_bounds__(256, gd16_waves(gd16_runs(AK, WMB), WMB * WNB)) void gemm16_direct_kernel(Gemm16Desc d) {
    static_assert(!AK || BK, "a k-major A comes with a k-major B");
    constexpr bool RUNS = gd16_runs(AK, WMB);
    constexpr int TM = 32 * WMB, TN = 32 * WNB;
    constexpr int LA = TM / 64, LB = TN / 64;        // load instructions per wave and step
    constexpr int SUB = (TM + TN) * 4, STAGE = KS * SUB;   // 16-byte slots of 32 k, of a stage
    constexpr int STEP_K = KS * G16_K;
    extern __shared__ u32x4 gd16_lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    int tile_x, tile_y, zz;
    gemm_tile_order(tile_x, tile_y, zz);
    const int m0 = tile_y * TM, n0 = tile_x * TN;
    const int split = zz % d.splits, z = zz / d.splits;
    const int z1 = z / d.inner, z2 = z - z1 * d.inner;
    const int k_begin = split * d.k_chunk;
    const int k_end = min(d.K, k_begin + d.k_chunk);
    const int steps = (k_end - k_begin + STEP_K - 1) / STEP_K;
    const bool tail = ((k_end - k_begin) % STEP_K) != 0;        // the last step is not a whole one

    // the operands advance one step per request; a segmented contraction jumps to the next segment's matrices
    const int seg0 = d.k_seg ? k_begin / d.k_seg : 0;
    int seg_left = d.k_seg ? d.k_seg - (k_begin - seg0 * d.k_seg) : 0x7fffffff;
    const int k_in_seg = d.k_seg ? k_begin - seg0 * d.k_seg : k_begin;
    const bf16_t* A = d.A + z1 * d.sa1 + z2 * d.sa2 + seg0 * d.sa_seg + (AK ? (int64_t)k_in_seg * d.lda + (m0 >> 5) * d.a_panel : (int64_t)m0 * d.lda + (k_in_seg >> 5) * d.a_panel);
    const bf16_t* B = d.B + z1 * d.sb1 + z2 * d.sb2 + seg0 * d.sb_seg + (BK ? (int64_t)k_in_seg * d.ldb + (n0 >> 5) * d.b_panel : (int64_t)n0 * d.ldb + (k_in_seg >> 5) * d.b_panel);
    const int64_t adv_a = AK ? (int64_t)G16_K * d.lda : d.a_panel, adv_b = BK ? (int64_t)G16_K * d.ldb : d.b_panel;
    uint32_t offa[LA], offb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        int row, k;
        gd16_slot<AK, false, TM>((4 * i + wave) * 64 + lane, row, k);
        if (AK) row = min(row, ((d.M - 1) & ~7) - m0);
        offa[i] = AK ? (uint32_t)(k * d.lda + (row >> 5) * (int)d.a_panel + (row & 31)) : (uint32_t)(min(row, d.M - 1 - m0) * d.lda + k);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        int row, k;
        gd16_slot<BK, true, TN>((4 * i + wave) * 64 + lane, row, k);
        if (BK) row = min(row, ((d.N - 1) & ~7) - n0);
        offb[i] = BK ? (uint32_t)(k * d.ldb + (row >> 5) * (int)d.b_panel + (row & 31)) : (uint32_t)(min(row, (EPI == 3 ? d.n_valid : d.N) - 1 - n0) * d.ldb + k);
    }
    auto load16 = [&](const bf16_t* src, u32x4* dst) {
        __builtin_amdgcn_global_load_lds((gd16_global_ptr*)src, (gd16_lds_ptr*)dst, 16, 0, 0);
    };
    auto advance = [&]() {
        A += KS * adv_a;
        B += KS * adv_b;
        seg_left -= STEP_K;
        if (seg_left == 0) {
            seg_left = d.k_seg;
            A += d.sa_seg - (AK ? (int64_t)d.k_seg * d.lda : (d.k_seg >> 5) * d.a_panel);
            B += d.sb_seg - (BK ? (int64_t)d.k_seg * d.ldb : (d.k_seg >> 5) * d.b_panel);
        }
    };
    auto request = [&](int step, int buf) {
#pragma unroll
        for (int sub = 0; sub < KS; ++sub) {
            u32x4* base = gd16_lds + buf * STAGE + sub * SUB;
            if (tail && step == steps - 1) {
                const int left = k_end - k_begin - step * STEP_K - sub * G16_K;   // below STEP_K - 32 sub; nothing of this part where it is not positive
#pragma unroll
                for (int i = 0; i < LA; ++i) {
                    int row, k;
                    gd16_slot<AK, false, TM>((4 * i + wave) * 64 + lane, row, k);
                    u32x4* dst = base + (4 * i + wave) * 64;
                    if (k < left) load16(A + sub * adv_a + offa[i], dst);
                    else dst[lane] = u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int i = 0; i < LB; ++i) {
                    int row, k;
                    gd16_slot<BK, true, TN>((4 * i + wave) * 64 + lane, row, k);
                    u32x4* dst = base + TM * 4 + (4 * i + wave) * 64;
                    if (k < left) load16(B + sub * adv_b + offb[i], dst);
                    else dst[lane] = u32x4{0u, 0u, 0u, 0u};
                }
                continue;
            }
#pragma unroll
            for (int i = 0; i < LA; ++i) load16(A + sub * adv_a + offa[i], base + (4 * i + wave) * 64);
#pragma unroll
            for (int i = 0; i < LB; ++i) load16(B + sub * adv_b + offb[i], base + TM * 4 + (4 * i + wave) * 64);
        }
        advance();
    };

    f32x4 acc[WMB][WNB];
#pragma unroll
    for (int i = 0; i < WMB; ++i)
#pragma unroll
        for (int j = 0; j < WNB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sum[RUNS ? WMB : 1][RUNS ? WNB : 1] = {};   // of the runs that are over
    // Operand reads; lane (r, g) holds k = 8g .. 8g + 7 of its row.  Block t of A: rows 16 t + r.  Row-major B: blocks 2p and
    // 2p + 1 are rows 32 p + 8 (r / 4) + r % 4 and four further, so that a lane's results of the two are eight neighbouring columns.
    // K-major: a transposing read takes a 4 (k) x 16 (rows) piece per 16 lanes, lane i of them at line i / 4, rows 4 (i % 4) ..;
    // two of them, lines 8g + i / 4 and four further, make the operand.  The 32-byte pieces of a line are permuted by the line
    // (gd16_slot), so that the eight lines that two neighbouring lane groups read together fall on different banks.
    const int piece = g ^ gd16_place(r >> 2);
    const int ra = (wm * 16 * WMB + r) * 4 + piece, rb = TM * 4 + (wn * 16 * WNB + 8 * (r >> 2) + (r & 3)) * 4 + piece;
    const int kline = 8 * g + (r >> 2);
    const int f128 = (r >> 2) | ((g & 1) << 2), f64 = (r >> 3) | ((g & 1) << 1);   // as in gd16_slot
    const int fa = TM >= 128 ? f128 : f64, fb = TN >= 128 ? f128 : f64;
    const int ta = kline * TM * 2 + 8 * (r & 3), tb = TM * 64 + kline * TN * 2 + 8 * (r & 3);   // bytes
    // One step out of LDS buffer `buf`; with LOAD it also requests a whole step into buffer `to`.  The order is fixed (the compiler's own
    // reads two blocks, waits for them, multiplies, and so on, and puts the loads in front): the operands of AHEAD block rows are
    // read first, those of the others AHEAD blocks before their use, and the load instructions, which the address unit takes 16
    // clocks each for, go out one by one between the matrix instructions.  Transposing reads come with their wait, so an AK step
    // reads all of them; its 256-row tile keeps the loads in front (32 000 x 512 over 8192 tokens: 226 us, 251 with the loads between).
    // 65 536 x 32 000 x 512 with statistics 2453 -> 2290 us, 8192 x 32 000 x 512 349 -> 307, 512 x 2048 over 8192 tokens 42 -> 38.
    auto multiply = [&](int buf, auto load, int to) {
        constexpr bool LOAD = decltype(load)::value, FRONT = AK && WMB >= 8;
        constexpr int AHEAD = !AK && WMB >= 8 ? 3 : WMB;
#pragma unroll
        for (int sub = 0; sub < KS; ++sub) {
            const u32x4* st = gd16_lds + buf * STAGE + sub * SUB;
            const uint32_t sb = (uint32_t)(uintptr_t)(gd16_lds_ptr*)st;
            u32x4* base = gd16_lds + to * STAGE + sub * SUB;
            auto piece = [&](int p) {
                if (p < LA) load16(A + sub * adv_a + offa[p], base + (4 * p + wave) * 64);
                else if (p < LA + LB) load16(B + sub * adv_b + offb[p - LA], base + TM * 4 + (4 * (p - LA) + wave) * 64);
            };
            u32x4 a[WMB], b[WNB];
            if constexpr (LOAD && FRONT)
#pragma unroll
                for (int p = 0; p < LA + LB; ++p) piece(p);
            if constexpr (!BK)
#pragma unroll
                for (int t = 0; t < WNB; ++t) b[t] = st[rb + 128 * (t >> 1) + 16 * (t & 1)];
            if constexpr (!AK)
#pragma unroll
                for (int t = 0; t < AHEAD; ++t) a[t] = st[ra + 64 * t];
            if constexpr (BK) {
                constexpr int NA = AK ? WMB : 0;
                uint32_t at[WNB + NA];
                u32x4 x[WNB + NA];
#pragma unroll
                for (int t = 0; t < WNB; ++t) at[t] = sb + tb + 32 * ((wn * WNB + t) ^ fb);
#pragma unroll
                for (int t = 0; t < NA; ++t) at[WNB + t] = sb + ta + 32 * ((wm * WMB + t) ^ fa);
                gd16_transposed<TN, TM, WNB, NA>(at, x);
#pragma unroll
                for (int t = 0; t < WNB; ++t) b[t] = x[t];
#pragma unroll
                for (int t = 0; t < NA; ++t) a[t] = x[WNB + t];
            }
            static_assert(LA + LB <= WMB, "a load per block row");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < WMB; ++mt) {
                if (!AK && mt + AHEAD < WMB) a[mt + AHEAD] = st[ra + 64 * (mt + AHEAD)];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_v, b[nt]), __builtin_bit_cast(bf16x8_v, a[mt]), acc[mt][nt], 0, 0, 0);
                if constexpr (LOAD && !FRONT) piece(mt);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (LOAD) advance();
    };
    auto end_of_run = [&](int i) {
        if constexpr (RUNS) {
            if ((i + 1) % (G16_RUN / KS) == 0) {
#pragma unroll
                for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                    for (int nt = 0; nt < WNB; ++nt) {
                        sum[mt][nt] += acc[mt][nt];
                        acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
        }
    };
#pragma unroll
    for (int i = 0; i < GD16_STAGES - 1; ++i)
        if (i < steps) request(i, i);
    int buf = 0, i = 0;
    // while whole steps are still to be requested; the GD16_STAGES - 2 youngest may stay in flight
    for (const int steady = steps - (GD16_STAGES - 1) - (tail ? 1 : 0); i < steady; ++i) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((GD16_STAGES - 2) * KS * (LA + LB)) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        multiply(buf, std::true_type{}, buf == 0 ? GD16_STAGES - 1 : buf - 1);
        buf = buf + 1 == GD16_STAGES ? 0 : buf + 1;
        end_of_run(i);
    }
    for (; i < steps; ++i) {
        // a tail is requested by fewer instructions: no counting with it
        if (!tail && i + 1 < steps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(KS * (LA + LB)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (i + GD16_STAGES - 1 < steps) request(i + GD16_STAGES - 1, buf == 0 ? GD16_STAGES - 1 : buf - 1);
        multiply(buf, std::false_type{}, 0);
        buf = buf + 1 == GD16_STAGES ? 0 : buf + 1;
        end_of_run(i);
    }
    if constexpr (RUNS)
#pragma unroll
        for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
            for (int nt = 0; nt < WNB; ++nt) acc[mt][nt] += sum[mt][nt];

    const bool plain = d.splits > 1;   // partial sums go out as they are; the reduction applies the epilogue
    const int64_t zoff = z1 * d.sc1 + z2 * d.sc2;
    float* C = plain ? d.part + ((int64_t)z * d.splits + split) * d.part_stride : d.C ? d.C + zoff : nullptr;
    const int64_t zoff16 = z1 * d.sc1_16 + z2 * d.sc2_16;
    bf16_t* C16 = (plain || !d.C16) ? nullptr : d.C16 + zoff16;
    bf16_t* G16 = (plain || !d.G16) ? nullptr : d.G16 + zoff16;
    const float* R = (plain || !d.R) ? nullptr : d.R + zoff;
    const float* bias = (plain || !d.bias) ? nullptr : d.bias + z1 * d.sbias1;
    const int ldc = plain ? d.N : d.ldc;
    const int m_base = m0 + wm * 16 * WMB, n_base = n0 + wn * 16 * WNB;
    if constexpr (EPI == 2) {
        if (d.alpha != 1.f)
#pragma unroll
            for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt) acc[mt][nt] *= d.alpha;
    }
    if constexpr (EPI == 3) {
        gd16_ce_grad<WMB, WNB>(d, acc, m_base, n_base, C16, r, g);
        return;
    }
    if constexpr (EPI == 4) gd16_gelu_bwd<WMB, WNB>(d, acc, m_base, n_base, 2 * tile_y + wm, r, g);
    const float alpha = EPI == 2 || EPI == 4 ? 1.f : d.alpha;   // above
    const bool vec = (plain ? (d.N & 3) == 0 : d.c_vec8 != 0) && m_base + 16 * WMB <= d.M && n_base + 16 * WNB <= d.N;
    if (EPI != 2 || C || C16) {
        if (vec) gd16_store<!BK, WMB, WNB, EPI == 1>(d, alpha, acc, m_base, n_base, C, C16, G16, R, bias, ldc, plain, r, g);
        else gd16_store_edge<!BK, WMB, WNB, EPI == 1>(d, alpha, acc, m_base, n_base, C, C16, G16, R, bias, ldc, plain, r, g);
    }
    if constexpr (EPI == 2) gd16_ce<WMB>(d, acc, m_base, n_base, 2 * tile_x + wn, r, g);   // leaves nothing of the block
}

// Rows of partial column sums that a product with gelu_part leaves: two per tile row
int gemm16_gelu_rows(int64_t M, int N) {
    const int64_t t84 = ((M + 255) / 256) * ((N + 127) / 128);
    return (int)(2 * (t84 >= 400 ? (M + 255) / 256 : (M + 127) / 128));
}

// Launch.  Split-K writes an fp32 output only and, with a batch, needs inner == 1; d.part must then hold
// batch*M*N*splits floats.
int launch_gemm16(hipStream_t s, Gemm16Desc d) {
    if (d.a_kmajor && !d.b_kmajor) return BLS_EUNSUPPORTED;   // no such product in this network
    if (d.splits < 1) d.splits = 1;
    if (d.inner < 1) d.inner = 1;
    if (d.batch < 1) d.batch = 1;
    int k_chunk = ((d.K + d.splits - 1) / d.splits + G16_K - 1) / G16_K * G16_K;
    d.splits = (d.K + k_chunk - 1) / k_chunk;
    d.k_chunk = k_chunk;
    d.part_stride = (int64_t)d.M * d.N;
    const bool panels = d.a_panel || d.b_panel;
    // row-major: the 32 columns of a step or of a block are 32 elements further
    if (d.a_panel == 0) d.a_panel = 32;
    else d.lda = 32;
    if (d.b_panel == 0) d.b_panel = 32;
    else d.ldb = 32;
    if (d.ldc16 == 0) {
        d.ldc16 = d.ldc;
        d.sc1_16 = d.sc1;
        d.sc2_16 = d.sc2;
    }
    if (d.c16_panel == 0) d.c16_panel = 32;
    auto al = [](const void* p, int bytes) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; };
    d.a_vec = (al(d.A, 16) && d.lda % 8 == 0 && d.sa1 % 8 == 0 && d.sa2 % 8 == 0) ? 1 : 0;
    d.b_vec = (al(d.B, 16) && d.ldb % 8 == 0 && d.sb1 % 8 == 0 && d.sb2 % 8 == 0) ? 1 : 0;
    d.c_vec = (al(d.C, 16) && al(d.R, 16) && al(d.bias, 16) && al(d.C16, 8) && al(d.G16, 8) && d.ldc % 4 == 0 && d.ldc16 % 4 == 0 && d.c16_panel % 4 == 0 && d.sc1_16 % 4 == 0 && d.sc2_16 % 4 == 0 && d.sc1 % 4 == 0 && d.sc2 % 4 == 0 && d.sbias1 % 4 == 0) ? 1 : 0;
    const bool half = d.C16 || d.G16;
    d.c_vec8 = (d.c_vec && al(d.C16, 16) && al(d.G16, 16) && (!half || (d.ldc16 % 8 == 0 && d.c16_panel % 8 == 0 && d.sc1_16 % 8 == 0 && d.sc2_16 % 8 == 0))) ? 1 : 0;
    // straight into LDS: 16-byte pieces of both factors (whole pieces along a contiguous K), 32-bit offsets inside a tile
    const bool direct = d.a_vec && d.b_vec && d.sa_seg % 8 == 0 && d.sb_seg % 8 == 0 && ((d.a_kmajor && d.b_kmajor) || (!d.a_kmajor && d.K % 8 == 0)) &&
                        (int64_t)256 * d.lda + 8 * d.a_panel < (int64_t(1) << 30) && (int64_t)256 * d.ldb + 8 * d.b_panel < (int64_t(1) << 30);
    if ((d.k_seg || d.ce_rows || d.gelu_part || panels) && !direct) return BLS_EUNSUPPORTED;   // gemm16_kernel takes none of the four
    if (direct) {
        const int z = d.batch * d.splits;
        const int64_t t84 = (int64_t)((d.M + 255) / 256) * ((d.N + 127) / 128) * z, t44 = (int64_t)((d.M + 127) / 128) * ((d.N + 127) / 128) * z;
        const int64_t t42 = (int64_t)((d.M + 127) / 128) * ((d.N + 63) / 64) * z;
        const bool deep = t42 <= 512 && d.k_seg % (2 * G16_K) == 0 && (d.splits == 1 || k_chunk % (2 * G16_K) == 0);
#define GD16_LAUNCH(AKM, BKM, EPI, WMB, WNB, KS)                                                                                     \
    hipLaunchKernelGGL((gemm16_direct_kernel<AKM, BKM, EPI, WMB, WNB, KS>),                                                               \
                       dim3((unsigned)((d.N + 32 * WNB - 1) / (32 * WNB)), (unsigned)((d.M + 32 * WMB - 1) / (32 * WMB)), z), dim3(256), \
                       GD16_STAGES * KS * 32 * (WMB + WNB) * 64, s, d)
#define GD16_TILE(AKM, BKM, EPI)                              \
    do {                                                      \
        if (t84 >= 400) GD16_LAUNCH(AKM, BKM, EPI, 8, 4, 1);     \
        else if (t44 >= 448) GD16_LAUNCH(AKM, BKM, EPI, 4, 4, 1); \
        else if (deep) GD16_LAUNCH(AKM, BKM, EPI, 4, 2, 2);    \
        else GD16_LAUNCH(AKM, BKM, EPI, 4, 2, 1);             \
    } while (0)
        // Tiles (measured, 8192 tokens): 256 x 128 from 400 of them (32 000 x 512 over the tokens, 500 tiles: 317 us, 364 with
        // 128 x 128); below that 128 x 128 from 448 (three 512-wide products: 23.2 us, 24.4 and 27.7 with the others); else
        // 128 x 64 (512 x 512: 14.4 us, 16.0 and 21.2).  A step of 32 is only 8 matrix instructions of a wave of that tile: where its
        // workgroups fit the chip two per compute unit (72 KB each), a step is 64 (512 x 512 over 8192 tokens in 8 parts 22.0 -> 19.6 us,
        // 8192 x 512 x 512 15.5 -> 14.7; 576 workgroups, a second round, 35 -> 38).
        if (d.ce_part) {   // statistics per 64 columns of a wave
            if (t84 >= 400) GD16_LAUNCH(false, false, 2, 8, 4, 1);
            else GD16_LAUNCH(false, false, 2, 4, 4, 1);
        } else if (d.ce_rows) {
            if (t84 >= 400) GD16_LAUNCH(false, false, 3, 8, 4, 1);
            else GD16_LAUNCH(false, false, 3, 4, 4, 1);
        } else if (d.gelu_part) {
            if (gemm16_gelu_rows(d.M, d.N) == 2 * ((d.M + 255) / 256)) GD16_LAUNCH(false, true, 4, 8, 4, 1);
            else GD16_LAUNCH(false, true, 4, 4, 4, 1);
        } else if (d.G16 && !d.a_kmajor && !d.b_kmajor) GD16_TILE(false, false, 1);
        else if (d.a_kmajor) GD16_TILE(true, true, 0);
        else if (d.b_kmajor) GD16_TILE(false, true, 0);
        else GD16_TILE(false, false, 0);
    } else {
        const dim3 grid((d.N + G16_TILE - 1) / G16_TILE, (d.M + G16_TILE - 1) / G16_TILE, d.batch * d.splits);
#define G16_LAUNCH(AKM, BKM, EPI) hipLaunchKernelGGL((gemm16_kernel<AKM, BKM, EPI>), grid, dim3(256), 0, s, d)
        if (d.ce_part) G16_LAUNCH(false, false, 2);   // row statistics: row-major factors, one matrix, no split
        else if (d.G16 && !d.b_kmajor) G16_LAUNCH(false, false, 1);
        else if (d.a_kmajor) G16_LAUNCH(true, true, 0);
        else if (d.b_kmajor) G16_LAUNCH(false, true, 0);
        else G16_LAUNCH(false, false, 0);
#undef G16_LAUNCH
    }
    if (d.splits > 1)
        launch_split_reduce(s, d.part, d.splits, d.M, d.N, d.batch, d.alpha, d.bias, d.sbias1, d.R, d.ldc, d.C, d.sc1, d.c_vec != 0);
    return BLS_OK;
}
