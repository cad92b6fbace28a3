// fp32 GEMM on the matrix cores for the sequence model: C[m][n] = alpha * sum_k A(m,k) B(n,k) [+ bias[n]] [+ R[m][n]].
//
// With G set the epilogue also stores gelu(C) there (erf form); C itself may then be NULL.
// A(m,k) is A[m*lda + k] or, with a_kmajor, A[k*lda + m]; likewise B(n,k).  With these two flags one kernel serves
// y = x W^T (both k-contiguous), dx = dy W (B k-major), dW = dy^T x (both k-major, contraction over tokens) and the
// attention products.  A batch index z = z1 * inner + z2 adds z1*s1 + z2*s2 to each base pointer (heads inside
// samples).  The contraction can be split over blockIdx.z into partial results that launch_split_reduce adds in split
// order (deterministic).
//
// Two kernels.  gemm_direct_kernel takes every product whose rows start on 16-byte boundaries: its tiles go from global
// memory straight into LDS.  gemm_tiled_kernel takes the others (odd pitches), element by element where it has to:
// 128 x 128 tile of C, four waves as 2 x 2, each 64 x 64 = 4 x 4 blocks of v_mfma_f32_16x16x4_f32; K advances 16 at a time
// through two LDS buffers holding As[k][m] and Bs[k][n] (row pitch 144 floats: a wave's read of 16 rows x 4 k-groups
// touches every bank exactly twice); the next step's global loads are in flight in registers meanwhile.
#include <limits.h>
#include <math.h>

#include "common.h"
#include "kernels.h"

#define GT_TILE 128
#define GT_K 16
#define GT_LD 144
#define GT_RUN 16   // steps in a running sum of a weight gradient

template <bool KMAJOR>
__device__ __forceinline__ void gt_fetch(const float* __restrict__ P, int ld, int rows, int K, int row0, int k0, int k_end, bool vec,
                                         f32x4 (&v)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int f = threadIdx.x + 256 * i;
        v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (KMAJOR) {
            const int k = k0 + (f >> 5), r = row0 + 4 * (f & 31);
            if (k < k_end) {
                const float* p = P + (int64_t)k * ld + r;
                if (vec && r + 3 < rows) v[i] = *reinterpret_cast<const f32x4*>(p);
                else
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (r + j < rows) v[i][j] = p[j];
            }
        } else {
            const int r = row0 + (f >> 2), k = k0 + 4 * (f & 3);
            if (r < rows) {
                const float* p = P + (int64_t)r * ld + k;
                if (vec && k + 3 < k_end) v[i] = *reinterpret_cast<const f32x4*>(p);
                else
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k + j < k_end) v[i][j] = p[j];
            }
        }
    }
    (void)K;
}

template <bool KMAJOR>
__device__ __forceinline__ void gt_put(float* __restrict__ S, const f32x4 (&v)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int f = threadIdx.x + 256 * i;
        if (KMAJOR) {
            *reinterpret_cast<f32x4*>(S + (f >> 5) * GT_LD + 4 * (f & 31)) = v[i];
        } else {
            const int r = f >> 2, k = 4 * (f & 3);
#pragma unroll
            for (int j = 0; j < 4; ++j) S[(k + j) * GT_LD + r] = v[i][j];
        }
    }
}

// Workgroups are handed to the eight XCDs (each with its own L2) round-robin in launch order.  When the tile count of
// one matrix divides by eight, launch slot i takes tile (i % 8) * (tiles / 8) + i / 8, so that an XCD walks a contiguous
// range of tiles, n fastest: the workgroups that share rows of A run on the same L2, one after the other.
__device__ __forceinline__ void gt_tile_of_block(int& tile_x, int& tile_y) {
    const int nx = gridDim.x, tiles = nx * gridDim.y;
    int id = blockIdx.y * nx + blockIdx.x;
    if ((tiles & 7) == 0) id = (id & 7) * (tiles >> 3) + (id >> 3);
    tile_y = id / nx;
    tile_x = id - tile_y * nx;
}

// Writes a wave's 64 x 64 block: lane (r, g) holds C[m = .. + 4g + i][n = .. + r] of every 16 x 16 block.  Blocks that
// lie inside C take the path without bounds checks.
template <bool GUARD>
__device__ __forceinline__ void gt_store_block(const GemmDesc& d, const f32x4 (&acc)[4][4], int m_base, int n_base, float* C, const float* R,
                                               const float* bias, int ldc, bool plain, int r, int g) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int n = n_base + nt * 16 + r;
            const float b = (bias && (!GUARD || n < d.N)) ? bias[n] : 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = m_base + mt * 16 + 4 * g + i;
                if (!GUARD || (m < d.M && n < d.N)) {
                    float v = acc[mt][nt][i];
                    if (!plain) {
                        v = v * d.alpha + b;
                        if (R) v += R[(int64_t)m * ldc + n];
                        if (d.G) d.G[(int64_t)m * ldc + n] = gelu_f32(v);
                    }
                    if (C) C[(int64_t)m * ldc + n] = v;
                }
            }
        }
}

__device__ __forceinline__ void gt_store(const GemmDesc& d, const f32x4 (&acc)[4][4], int m_base, int n_base, int z, int z1, int z2, int split,
                                         int r, int g) {
    const bool plain = d.splits > 1;   // partial sums go out as they are; the reduction applies the epilogue
    float* C = plain ? d.part + ((int64_t)z * d.splits + split) * d.part_stride : d.C ? d.C + z1 * d.sc1 + z2 * d.sc2 : nullptr;
    const int ldc = plain ? d.N : d.ldc;
    const float* R = (plain || !d.R) ? nullptr : d.R + z1 * d.sc1 + z2 * d.sc2;
    const float* bias = (plain || !d.bias) ? nullptr : d.bias + z1 * d.sbias1;
    if (m_base + 64 <= d.M && n_base + 64 <= d.N) gt_store_block<false>(d, acc, m_base, n_base, C, R, bias, ldc, plain, r, g);
    else gt_store_block<true>(d, acc, m_base, n_base, C, R, bias, ldc, plain, r, g);
}

template <bool AK, bool BK>
__global__ __launch_bounds__(256) void gemm_tiled_kernel(GemmDesc d) {
    __shared__ float As[2][GT_K * GT_LD], Bs[2][GT_K * GT_LD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    int tile_x, tile_y;
    gt_tile_of_block(tile_x, tile_y);
    const int m0 = tile_y * GT_TILE, n0 = tile_x * GT_TILE;
    const int split = blockIdx.z % d.splits, z = blockIdx.z / d.splits;
    const int z1 = z / d.inner, z2 = z - z1 * d.inner;
    const float* A = d.A + z1 * d.sa1 + z2 * d.sa2;
    const float* B = d.B + z1 * d.sb1 + z2 * d.sb2;
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

    f32x4 pa[2], pb[2];
    gt_fetch<AK>(A, d.lda, d.M, d.K, m0, k_begin, k_end, avec, pa);
    gt_fetch<BK>(B, d.ldb, d.N, d.K, n0, k_begin, k_end, bvec, pb);
    gt_put<AK>(As[0], pa);
    gt_put<BK>(Bs[0], pb);
    __syncthreads();
    int buf = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += GT_K) {
        const bool more = k0 + GT_K < k_end;
        if (more) {
            gt_fetch<AK>(A, d.lda, d.M, d.K, m0, k0 + GT_K, k_end, avec, pa);
            gt_fetch<BK>(B, d.ldb, d.N, d.K, n0, k0 + GT_K, k_end, bvec, pb);
        }
        const float* as = As[buf] + wm * 64 + r;
        const float* bs = Bs[buf] + wn * 64 + r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float a[4], b[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                a[t] = as[(4 * j + g) * GT_LD + 16 * t];
                b[t] = bs[(4 * j + g) * GT_LD + 16 * t];
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mt], b[nt], acc[mt][nt], 0, 0, 0);
        }
        if (more) {
            gt_put<AK>(As[buf ^ 1], pa);
            gt_put<BK>(Bs[buf ^ 1], pb);
        }
        if constexpr (AK)
            if (++in_run == GT_RUN) {
                in_run = 0;
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt) {
                        sum[mt][nt] += acc[mt][nt];
                        acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
        __syncthreads();
        buf ^= 1;
    }
    if constexpr (AK)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) acc[mt][nt] += sum[mt][nt];
    gt_store(d, acc, m0 + wm * 64, n0 + wn * 64, z, z1, z2, split, r, g);
}

// ---- tiles straight into LDS -------------------------------------------------------------------------------------------
//
// Workgroup = 32 WMB x 32 WNB tile of C, four waves as 2 x 2, each 16 WMB x 16 WNB.  K advances GT_K = 16 at a time
// through GD_STAGES LDS buffers that global_load_lds fills (16 bytes per lane, the 64 lanes of an instruction fill 1 KB of
// consecutive LDS): no staging registers, and GD_STAGES - 1 steps of loads in flight however long the matrix instructions
// of a step take.  One barrier per step: a wave waits for its own loads of the step (counted, the younger steps stay in
// flight), the barrier makes everybody's visible and frees the buffer that was read a step ago.
//
// LDS layout.  A row-major operand is [row][16 k]: lane (r, g) reads k = 4g .. 4g + 3 of row r with one 16-byte read that
// feeds four matrix instructions, instruction j taking k = 4g + j (the order of k inside a step is free as long as both
// operands agree).  Rows are 64 bytes, so the 16-byte pieces of a row are permuted, piece c to place c ^ ((row / 4) % 4): a
// read of 16 rows then covers all 64 banks.  A k-major operand is [k][row], read 4 bytes at a time; piece c (4 rows) of line
// k sits at place c ^ 4 (k / 4 % 4), which spreads the four lane groups of a read.  The permutation costs nothing: it is the
// lane that fetches another address.
//
// Rows past the end of an operand are clamped to the last one (they only feed outputs that are never stored); pieces past the
// end of K are zeroed in LDS in the last step.
//
// Tile choice (launcher): the tile for which the busiest compute unit has least to do.  3100 tokens x 512 outputs are 100
// tiles of 128 x 128 for 256 compute units but 196 of 64 x 128.
//
// Both operands k-major: a weight gradient, whose contraction runs over all tokens.  Its sums are taken in runs of GT_RUN steps,
// whatever tile and split the launcher takes: one running sum over 3100 tokens left the gradient of a 2048 x 512 layer 8.3e-7 off
// (relative 2-norm), runs of 256 leave 1.2e-7.  Two steps of 31 x 100 tokens on the 6-layer encoder: 16.00 -> 16.08 ms (the
// 128 x 128 tile keeps two workgroups per compute unit instead of three).
#define GD_STAGES 3
typedef __attribute__((address_space(1))) const void gd_global_ptr;
typedef __attribute__((address_space(3))) void gd_lds_ptr;

// Slot v (16 bytes) of an operand stage of ROWS rows: the piece of the matrix that belongs there.
template <bool KMAJOR, int ROWS>
__device__ __forceinline__ void gd_slot(int v, int& row, int& k) {
    if (KMAJOR) {
        constexpr int CPR = ROWS / 4;
        k = v / CPR;
        row = 4 * ((v % CPR) ^ (4 * ((k >> 2) & 3)));
    } else {
        row = v >> 2;
        k = 4 * ((v & 3) ^ ((row >> 2) & 3));
    }
}

template <bool AK, bool BK, int WMB, int WNB>
__global__ __launch_bounds__(256, 2) void gemm_direct_kernel(GemmDesc d) {
    static_assert(!AK || BK, "a k-major A comes with a k-major B");
    constexpr int TM = 32 * WMB, TN = 32 * WNB;
    constexpr int LA = TM / 64, LB = TN / 64;                 // load instructions per wave and step
    constexpr int STAGE = (TM + TN) * GT_K;                   // floats
    extern __shared__ f32x4 gd_lds[];
    float* lds = reinterpret_cast<float*>(gd_lds);
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
    const int steps = (k_end - k_begin + GT_K - 1) / GT_K;
    const bool tail = ((k_end - k_begin) % GT_K) != 0;        // the last step is not a whole one

    // The operands advance one step per request; a segmented contraction jumps to the next segment's matrices.
    const int seg0 = d.k_seg ? k_begin / d.k_seg : 0;
    int seg_left = d.k_seg ? d.k_seg - (k_begin - seg0 * d.k_seg) : INT_MAX;
    const int k_in_seg = d.k_seg ? k_begin - seg0 * d.k_seg : k_begin;
    const float* A = d.A + z1 * d.sa1 + z2 * d.sa2 + seg0 * d.sa_seg + (AK ? (int64_t)k_in_seg * d.lda + m0 : (int64_t)m0 * d.lda + k_in_seg);
    const float* B = d.B + z1 * d.sb1 + z2 * d.sb2 + seg0 * d.sb_seg + (BK ? (int64_t)k_in_seg * d.ldb + n0 : (int64_t)n0 * d.ldb + k_in_seg);
    const int64_t adv_a = AK ? (int64_t)GT_K * d.lda : GT_K, adv_b = BK ? (int64_t)GT_K * d.ldb : GT_K;
    uint32_t offa[LA], offb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        int row, k;
        gd_slot<AK, TM>((4 * i + wave) * 64 + lane, row, k);
        offa[i] = AK ? (uint32_t)(k * d.lda + min(row, ((d.M - 1) & ~3) - m0)) : (uint32_t)(min(row, d.M - 1 - m0) * d.lda + k);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        int row, k;
        gd_slot<BK, TN>((4 * i + wave) * 64 + lane, row, k);
        offb[i] = BK ? (uint32_t)(k * d.ldb + min(row, ((d.N - 1) & ~3) - n0)) : (uint32_t)(min(row, d.N - 1 - n0) * d.ldb + k);
    }
    auto load16 = [&](const float* src, int slot) {
        __builtin_amdgcn_global_load_lds((gd_global_ptr*)src, (gd_lds_ptr*)(lds + 4 * slot), 16, 0, 0);
    };
    // request of step `step` (they come in order) into buffer `buf`
    auto request = [&](int step, int buf) {
        const int base = buf * (STAGE / 4);
        if (tail && step == steps - 1) {
            const int left = k_end - k_begin - step * GT_K;   // 1 .. 15
#pragma unroll
            for (int i = 0; i < LA; ++i) {
                int row, k;
                const int v = (4 * i + wave) * 64 + lane;
                gd_slot<AK, TM>(v, row, k);
                if (k < left) load16(A + offa[i], base + (4 * i + wave) * 64);
                else gd_lds[base + v] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < LB; ++i) {
                int row, k;
                const int v = (4 * i + wave) * 64 + lane;
                gd_slot<BK, TN>(v, row, k);
                if (k < left) load16(B + offb[i], base + TM * 4 + (4 * i + wave) * 64);
                else gd_lds[base + TM * 4 + v] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < LA; ++i) load16(A + offa[i], base + (4 * i + wave) * 64);
#pragma unroll
        for (int i = 0; i < LB; ++i) load16(B + offb[i], base + TM * 4 + (4 * i + wave) * 64);
        A += adv_a;
        B += adv_b;
        seg_left -= GT_K;
        if (seg_left == 0) {
            seg_left = d.k_seg;
            A += d.sa_seg - (AK ? (int64_t)d.k_seg * d.lda : (int64_t)d.k_seg);
            B += d.sb_seg - (BK ? (int64_t)d.k_seg * d.ldb : (int64_t)d.k_seg);
        }
    };

    f32x4 acc[WMB][WNB];
#pragma unroll
    for (int i = 0; i < WMB; ++i)
#pragma unroll
        for (int j = 0; j < WNB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sum[AK ? WMB : 1][AK ? WNB : 1] = {};   // of the runs that are over

    // float offsets of the lane's operands in a stage
    int ra, rb;   // row-major: the 16-byte piece of row r of block 0; k-major: see below
    ra = AK ? 0 : (wm * 16 * WMB + r) * GT_K + 4 * (g ^ ((r >> 2) & 3));
    rb = BK ? 0 : (wn * 16 * WNB + r) * GT_K + 4 * (g ^ ((r >> 2) & 3));
    auto compute = [&](int buf) {
        const float* as = lds + buf * STAGE;
        const float* bs = as + TM * GT_K;
        f32x4 a[WMB], b[WNB];
        if (!AK)
#pragma unroll
            for (int t = 0; t < WMB; ++t) a[t] = *reinterpret_cast<const f32x4*>(as + ra + 16 * t * GT_K);
        if (!BK)
#pragma unroll
            for (int t = 0; t < WNB; ++t) b[t] = *reinterpret_cast<const f32x4*>(bs + rb + 16 * t * GT_K);
        // k-major: row 16 t + r of line k = 4 g + j; the pieces of 16 rows (4 of them) move together: block t to t ^ g
        if (AK)
#pragma unroll
            for (int t = 0; t < WMB; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) a[t][j] = as[(4 * g + j) * TM + 16 * ((wm * WMB + t) ^ g) + r];
        if (BK)
#pragma unroll
            for (int t = 0; t < WNB; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) b[t][j] = bs[(4 * g + j) * TN + 16 * ((wn * WNB + t) ^ g) + r];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt) acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[nt][j], a[mt][j], acc[mt][nt], 0, 0, 0);
    };

#pragma unroll
    for (int i = 0; i < GD_STAGES - 1; ++i)
        if (i < steps) request(i, i);
    int buf = 0;
    for (int i = 0; i < steps; ++i) {
        // while a later step is still to be requested the GD_STAGES - 2 youngest steps may stay in flight
        if (i + GD_STAGES - 1 < steps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((GD_STAGES - 2) * (LA + LB)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (i + GD_STAGES - 1 < steps) request(i + GD_STAGES - 1, buf == 0 ? GD_STAGES - 1 : buf - 1);
        compute(buf);
        buf = buf + 1 == GD_STAGES ? 0 : buf + 1;
        if constexpr (AK) {
            if ((i + 1) % GT_RUN == 0) {
#pragma unroll
                for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                    for (int nt = 0; nt < WNB; ++nt) {
                        sum[mt][nt] += acc[mt][nt];
                        acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
        }
    }
    if constexpr (AK)
#pragma unroll
        for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
            for (int nt = 0; nt < WNB; ++nt) acc[mt][nt] += sum[mt][nt];

    // lane (r, g) holds acc[mt][nt][i] = C[.. + r][.. + 4g + i] of every 16 x 16 block
    const bool plain = d.splits > 1;   // partial sums go out as they are; the reduction applies the epilogue
    float* C = plain ? d.part + ((int64_t)z * d.splits + split) * d.part_stride : d.C ? d.C + z1 * d.sc1 + z2 * d.sc2 : nullptr;
    const int ldc = plain ? d.N : d.ldc;
    const float* R = (plain || !d.R) ? nullptr : d.R + z1 * d.sc1 + z2 * d.sc2;
    const float* bias = (plain || !d.bias) ? nullptr : d.bias + z1 * d.sbias1;
    const bool vec = plain ? (d.N & 3) == 0 : d.c_vec != 0;
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m0 + (wm * WMB + mt) * 16 + r;
        if (m >= d.M) continue;
#pragma unroll
        for (int nt = 0; nt < WNB; ++nt) {
            const int n = n0 + (wn * WNB + nt) * 16 + 4 * g;
            if (n >= d.N) continue;
            const int64_t at = (int64_t)m * ldc + n;
            f32x4 v = acc[mt][nt];
            if (vec && n + 3 < d.N) {
                if (!plain) {
                    v *= d.alpha;
                    if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
                    if (R) v += *reinterpret_cast<const f32x4*>(R + at);
                    if (d.G) {
                        f32x4 q;
#pragma unroll
                        for (int i = 0; i < 4; ++i) q[i] = gelu_f32(v[i]);
                        *reinterpret_cast<f32x4*>(d.G + at) = q;
                    }
                }
                if (C) *reinterpret_cast<f32x4*>(C + at) = v;
            } else {
                for (int i = 0; i < 4 && n + i < d.N; ++i) {
                    float q = v[i];
                    if (!plain) {
                        q *= d.alpha;
                        if (bias) q += bias[n + i];
                        if (R) q += R[at + i];
                        if (d.G) d.G[at + i] = gelu_f32(q);
                    }
                    if (C) C[at + i] = q;
                }
            }
        }
    }
}

// out[i] = alpha * sum_z part[z][i] (+ bias) (+ R), in split order; blockIdx.y is the matrix of a batch (outer index only)
__global__ __launch_bounds__(256) void gemm_split_reduce_kernel(const float* __restrict__ part, int splits, int M, int N, float alpha,
                                                                const float* __restrict__ bias, const float* __restrict__ R, int ldc,
                                                                float* __restrict__ out, int64_t sc1, int64_t sbias1) {
    const int64_t total = (int64_t)M * N;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    part += (int64_t)blockIdx.y * splits * total;
    out += (int64_t)blockIdx.y * sc1;
    if (R) R += (int64_t)blockIdx.y * sc1;
    if (bias) bias += (int64_t)blockIdx.y * sbias1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        float acc = part[i];
        for (int zz = 1; zz < splits; ++zz) acc += part[(int64_t)zz * total + i];
        const int64_t m = i / N;
        const int n = (int)(i - m * N);
        acc *= alpha;
        if (bias) acc += bias[n];
        if (R) acc += R[m * ldc + n];
        out[m * ldc + n] = acc;
    }
}
// The same four columns at a time: N % 4 == 0 and 16-byte aligned rows everywhere
__global__ __launch_bounds__(256) void gemm_split_reduce4_kernel(const f32x4* __restrict__ part, int splits, int M, int N4, float alpha,
                                                                 const float* __restrict__ bias, const float* __restrict__ R, int ldc,
                                                                 float* __restrict__ out, int64_t sc1, int64_t sbias1) {
    const int64_t total = (int64_t)M * N4;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    part += (int64_t)blockIdx.y * splits * total;
    out += (int64_t)blockIdx.y * sc1;
    if (R) R += (int64_t)blockIdx.y * sc1;
    if (bias) bias += (int64_t)blockIdx.y * sbias1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        f32x4 acc = part[i];
#pragma unroll 4
        for (int zz = 1; zz < splits; ++zz) acc += part[(int64_t)zz * total + i];
        const int64_t m = i / N4;
        const int n = 4 * (int)(i - m * N4);
        acc *= alpha;
        if (bias) acc += *reinterpret_cast<const f32x4*>(bias + n);
        if (R) acc += *reinterpret_cast<const f32x4*>(R + m * ldc + n);
        *reinterpret_cast<f32x4*>(out + m * ldc + n) = acc;
    }
}

// `aligned`: bias, R and out allow 16-byte accesses in every row
void launch_split_reduce(hipStream_t s, const float* part, int splits, int M, int N, int batch, float alpha, const float* bias, int64_t sbias1,
                         const float* R, int ldc, float* out, int64_t sc1, bool aligned) {
    const bool vec = N % 4 == 0 && aligned;
    int64_t blocks = ceil_div((int64_t)M * N / (vec ? 4 : 1), 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    if (vec)
        hipLaunchKernelGGL(gemm_split_reduce4_kernel, dim3((unsigned)blocks, batch), dim3(256), 0, s, reinterpret_cast<const f32x4*>(part), splits, M,
                           N / 4, alpha, bias, R, ldc, out, sc1, sbias1);
    else
        hipLaunchKernelGGL(gemm_split_reduce_kernel, dim3((unsigned)blocks, batch), dim3(256), 0, s, part, splits, M, N, alpha, bias, R, ldc, out, sc1,
                           sbias1);
}

size_t gemm_tiled_partial_floats(int M, int N, int splits) { return splits > 1 ? (size_t)M * N * splits : 0; }

// Tile and split of a product on gemm_direct_kernel: the pair with the smallest estimate of
//   (rounds of workgroups over the compute units) x (K steps of a workgroup + six for its first loads and epilogue) x (time
//   of a step) + the pass that adds the partial sums.
// A step of a 16 x 16 block is 8192 flop, 13.3 ns of a compute unit's matrix pipes; the factors on it are what the tiles
// reach on large products.
struct GdPlan {
    int wmb, wnb, splits;
};
static GdPlan gd_plan(int64_t M, int64_t N, int64_t K, int batch, int max_splits) {
    static const struct { int wmb, wnb; double step; } tiles[3] = {{4, 4, 1.15}, {2, 4, 1.25}, {2, 2, 1.4}};
    GdPlan best{4, 4, 1};
    double best_us = 1e30;
    for (const auto& t : tiles)
        for (int sp = 1; sp <= max_splits; ++sp) {
            if (sp > 1 && K / sp < 8 * GT_K) break;
            const double wgs = (double)ceil_div(M, 32 * t.wmb) * (double)ceil_div(N, 32 * t.wnb) * batch * sp;
            const double steps = (double)ceil_div(ceil_div(K, sp), GT_K) + 6.0;
            double us = ceil(wgs / 256.0) * steps * 4 * t.wmb * t.wnb * t.step * 0.0133;
            if (sp > 1) us += 3.0 + (sp + 1.0) * (double)M * (double)N * batch * 4.0 / 4.0e6;
            if (us < best_us) {
                best_us = us;
                best = GdPlan{t.wmb, t.wnb, sp};
            }
        }
    return best;
}

template <bool AK, bool BK>
static void launch_direct(hipStream_t s, const GemmDesc& d, const GdPlan& p) {
    const int z = d.batch * d.splits;
#define GD_LAUNCH(WMB, WNB)                                                                                                            \
    hipLaunchKernelGGL((gemm_direct_kernel<AK, BK, WMB, WNB>), dim3((unsigned)ceil_div(d.N, 32 * WNB), (unsigned)ceil_div(d.M, 32 * WMB), z), \
                       dim3(256), GD_STAGES * 32 * (WMB + WNB) * GT_K * (int)sizeof(float), s, d)
    if (p.wmb == 4) GD_LAUNCH(4, 4);
    else if (p.wnb == 4) GD_LAUNCH(2, 4);
    else GD_LAUNCH(2, 2);
#undef GD_LAUNCH
}

// Launch.  Split-K with a batch needs inner == 1; d.part must then hold batch*M*N*splits floats.
int launch_gemm_tiled(hipStream_t s, GemmDesc d) {
    if (d.a_kmajor && !d.b_kmajor) return BLS_EUNSUPPORTED;   // no such product in this network
    if (d.splits < 1) d.splits = 1;
    if (d.inner < 1) d.inner = 1;
    if (d.batch < 1) d.batch = 1;
    auto aligned = [](const float* p, int ld, int64_t s1, int64_t s2, int64_t s3) {
        return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 4 == 0 && s1 % 4 == 0 && s2 % 4 == 0 && s3 % 4 == 0;
    };
    d.a_vec = aligned(d.A, d.lda, d.sa1, d.sa2, d.sa_seg) ? 1 : 0;
    d.b_vec = aligned(d.B, d.ldb, d.sb1, d.sb2, d.sb_seg) ? 1 : 0;
    d.c_vec = aligned(d.C, d.ldc, d.sc1, d.sc2, d.sbias1) && aligned(d.R, 0, 0, 0, 0) && aligned(d.bias, 0, 0, 0, 0) && aligned(d.G, 0, 0, 0, 0) ? 1 : 0;
    // straight into LDS: 16-byte pieces of both operands, whole pieces along K, 32-bit offsets inside a tile's rows
    const bool direct = d.a_vec && d.b_vec && ((d.a_kmajor && d.b_kmajor) || d.K % 4 == 0) && (int64_t)128 * d.lda < (int64_t(1) << 29) &&
                        (int64_t)128 * d.ldb < (int64_t(1) << 29);
    if (d.k_seg && !direct) return BLS_EUNSUPPORTED;   // gemm_tiled_kernel reads one pair of matrices
    GdPlan plan{4, 4, d.splits};
    if (direct) plan = gd_plan(d.M, d.N, d.K, d.batch, d.splits);
    // A contraction of up to eight steps is latency: workgroups of the smallest tile, of which more run side by side, beat the plan at
    // every size (scores of 64 / 1500 sequences of 100 / 128 tokens, width 128, plan and smallest tile: 248 / 220 us, 4.32 / 4.08 ms; width 64, 256 sequences 347 / 326
    // us; training 31 x 100 tokens, width 512, two layers 2.81 / 2.74 ms).  Contractions of one or two steps store more than they multiply, so from four
    // workgroups per compute unit on the plan decides there (8192 tokens x 32 000 words, widths 16 and 32: scores 585 / 622 and 655 / 676 us).
    if (direct && plan.splits == 1 && d.K <= 8 * GT_K &&
        (d.K > 2 * GT_K || (int64_t)d.batch * ceil_div(d.M, 64) * ceil_div(d.N, 64) <= 1024))
        plan = GdPlan{2, 2, 1};
    const int k_chunk = (int)ceil_div(ceil_div(d.K, plan.splits), GT_K) * GT_K;
    d.splits = (int)ceil_div(d.K, k_chunk);
    d.k_chunk = k_chunk;
    d.part_stride = (int64_t)d.M * d.N;
    if (direct) {
        if (d.a_kmajor) launch_direct<true, true>(s, d, plan);
        else if (d.b_kmajor) launch_direct<false, true>(s, d, plan);
        else launch_direct<false, false>(s, d, plan);
    } else {
        dim3 grid((d.N + GT_TILE - 1) / GT_TILE, (d.M + GT_TILE - 1) / GT_TILE, d.batch * d.splits);
        if (d.a_kmajor) hipLaunchKernelGGL((gemm_tiled_kernel<true, true>), grid, dim3(256), 0, s, d);
        else if (d.b_kmajor) hipLaunchKernelGGL((gemm_tiled_kernel<false, true>), grid, dim3(256), 0, s, d);
        else hipLaunchKernelGGL((gemm_tiled_kernel<false, false>), grid, dim3(256), 0, s, d);
    }
    if (d.splits > 1)
        launch_split_reduce(s, d.part, d.splits, d.M, d.N, d.batch, d.alpha, d.bias, d.sbias1, d.R, d.ldc, d.C, d.sc1, d.c_vec != 0);
    return BLS_OK;
}
