// fp32 products of the sequence model's training steps on the bf16 matrix instructions, without giving up fp32 precision:
// C[m][n] = alpha * sum_k A(m,k) B(n,k) [+ bias[n]] [+ R[m][n]], A as in gemm_tiled.hip, B packed (below).
//
// Every fp32 value is the exact sum of three bf16 values, h + m + l (3 x 8 bits; h is x rounded, m what is left rounded, l the
// rest).  Of the nine partial products six are summed (l h, h l, m m, m h, h m, h h); the three left out, m l, l m and l l, are at most
// 2^-24 of a product together, 2^-27.5 in the mean square.  Six bf16 instructions take 3/8 of the matrix-pipe time of the fp32
// instructions for the same block, and round less often: the h h products have an accumulator of their own (one rounding per 16
// values of k instead of four per 16), the others, 2^-8 of its size, a second one.  Relative 2-norm error against 64 bits, normal factors,
// contraction of 16 / 32 / 64 / 512 / 2048 / 32 000: fp32 instruction 7.4e-8 / 1.0e-7 / 1.4e-7 / 4.0e-7 / 8.1e-7 / 3.2e-6, this 3.2e-8 / 3.9e-8 / 5.0e-8 /
// 1.3e-7 / 2.7e-7 / 1.1e-6; one accumulator for all six would be at 3.3e-7 for 512 and biased (the instruction truncates towards minus
// infinity).  Where one product of a sum dwarfs the others that truncation is what is left, and the fp32 instruction is closer: factors
// spread log-normally over e^3, 16 / 64 / 2048 values 2.6e-8 / 7.0e-8 / 1.1e-7, this 4.1e-8 / 8.2e-8 / 1.3e-7 (gradients of encoders: half its
// error in the median, a third in the worst tensor).  Weight gradients (A k-major) fold the first accumulator every GT_RUN steps: 3100 tokens
// 1.1e-7, fp32 instructions in the same runs 2.9e-7.
// Values below 2^-110 lose the bits of l and m that bf16 cannot hold (2^-133).
//
// Infinities, NaN and values that round to a bf16 infinity: h + m + l is NaN or infinity minus infinity there, and h h may be beyond
// the largest float where the product is not (h is up to 2^-8 above its factor), so a result that is not finite is the sign; the
// workgroup then does its contraction again with the fp32 instruction (whose results are those of fp32 arithmetic: an infinite factor
// gives an infinite result).
//
// What bounds it is the vector unit beside the matrix pipe: splitting takes 5.5 vector instructions a value, and a SIMD that runs
// 8 of them per matrix instruction (two waves, interleaved as well as it goes) reaches 70 % of its matrix rate, with 4 it reaches all
// of it; a wave that is alone on its SIMD issues one vector instruction in 6 to 7 cycles.  With both operands split on the way from
// LDS (7.3 per matrix instruction) 3100 x 32 000 x 512 took 631 us (fp32 instructions: 855).  So B comes split from memory, 560 us:
// split_pack_kernel writes the weights once per step, in both orders, and the second factor of a weight gradient before its product.
// Large products run the matrix pipes 55 to 63 % of the time at 1.8 GHz (power), 160 to 185 Tflop/s of fp32 work; 3100 x 512 x 2048
// has too few tiles for that (50 us; 75 with fp32 instructions).  Reading and splitting the next step between the matrix
// instructions of this one (57 us against 62 for one workgroup per compute unit, 612 against 560 us for the large one, 100
// registers more) and deeper load queues (no change) were taken back; dot products that subtract the bf16 parts (3.5 instructions
// a value) run on the matrix pipe themselves.
//
// Pack of a matrix B(n,k), N rows: [k / 16][plane h, m, l][k / 8 % 2][n][k % 8], zeros where k is past the end.  What a step of 16
// needs of 64 rows is six stretches of 1 KB, which is what one global_load_lds of a wave moves, and the 32 rows that half a wave
// reads are 512 consecutive bytes of LDS.
#include <limits.h>
#include <math.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

#define GS_K 16
#define GT_RUN 16   // steps in a running sum of a weight gradient

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const void gs_global_ptr;
typedef __attribute__((address_space(3))) void gs_lds_ptr;

struct Split8 {   // eight values: pairs of bf16
    uint32_t h[4], m[4], l[4];
};
__device__ __forceinline__ bf16x8 bf16x8_of(const uint32_t (&v)[4]) { return __builtin_bit_cast(bf16x8, u32x4{v[0], v[1], v[2], v[3]}); }
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
}
__device__ __forceinline__ Split8 split8(f32x4 lo, f32x4 hi) {
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x4 v = i < 2 ? lo : hi;
        float x = v[2 * (i & 1)], y = v[2 * (i & 1) + 1];
        s.h[i] = bf16_pair(x, y);
        x -= __uint_as_float(s.h[i] << 16);
        y -= __uint_as_float(s.h[i] & 0xffff0000u);
        s.m[i] = bf16_pair(x, y);
        x -= __uint_as_float(s.m[i] << 16);
        y -= __uint_as_float(s.m[i] & 0xffff0000u);
        s.l[i] = bf16_pair(x, y);
    }
    return s;
}

// ---- packs -----------------------------------------------------------------------------------------------------------

// One value, exactly, whatever it is: a finite value that rounds to infinity is cut instead, infinities and NaN are h alone.
__device__ __forceinline__ void split_any(float x, uint32_t& h, uint32_t& m, uint32_t& l) {
    const uint32_t u = __float_as_uint(x);
    const bool finite = (u & 0x7f800000u) != 0x7f800000u;
    h = bf16_pair(x, 0.f) & 0xffffu;
    if (finite && (h & 0x7f80u) == 0x7f80u) h = u >> 16;
    const float r = finite ? x - __uint_as_float(h << 16) : 0.f;
    m = bf16_pair(r, 0.f) & 0xffffu;
    l = bf16_pair(r - __uint_as_float(m << 16), 0.f) & 0xffffu;
}
__device__ __forceinline__ void store_pack(uint16_t* __restrict__ dst, int64_t rows, int k8, int64_t n, const float (&v)[8]) {
    uint32_t p[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t a[3], b[3];
        split_any(v[2 * i], a[0], a[1], a[2]);
        split_any(v[2 * i + 1], b[0], b[1], b[2]);
#pragma unroll
        for (int j = 0; j < 3; ++j) p[j][i] = a[j] | (b[j] << 16);
    }
    const int64_t step = k8 >> 1, half = k8 & 1;
#pragma unroll
    for (int j = 0; j < 3; ++j)
        *reinterpret_cast<u32x4*>(dst + ((step * 6 + 2 * j + half) * rows + n) * 8) = u32x4{p[j][0], p[j][1], p[j][2], p[j][3]};
}

// Memory bound: four bytes read and six written a value.  A k-major source (x[k][n]) is read and written in whole lines: a thread
// takes one n and 16 values of k.  A row-major one (x[n][k]): eight adjacent threads read 256 bytes of a row, eight rows of a
// wave write 128 bytes of a plane.
template <bool KMAJOR>
__global__ __launch_bounds__(256) void split_pack_kernel(SplitPackTable tab, const float* __restrict__ src, uint16_t* __restrict__ dst) {
    int j = 0, b = blockIdx.x;
    while (j + 1 < tab.n && b >= tab.j[j].blocks) b -= tab.j[j++].blocks;
    const SplitPackJob job = tab.j[j];
    src += job.src;
    dst += job.dst;
    float v[8];
    if (KMAJOR) {
        const int nb = (job.rows + 255) >> 8;
        const int step = b / nb, n = (b - step * nb) * 256 + threadIdx.x;
        if (n >= job.rows) return;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int k0 = step * GS_K + 8 * half;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = k0 + i < job.K ? src[(int64_t)(k0 + i) * job.ld + n] : 0.f;
            store_pack(dst, job.rows, 2 * step + half, n, v);
        }
    } else {
        const int kb = (job.K + 63) >> 6;
        const int rb = b / kb, k0 = (b - rb * kb) * 64 + 8 * (threadIdx.x & 7);
        if (k0 >= (job.K + GS_K - 1) / GS_K * GS_K) return;
        const bool vec = (job.ld & 3) == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int n = rb * 64 + 32 * it + (threadIdx.x >> 3);
            if (n >= job.rows) return;
            const float* p = src + (int64_t)n * job.ld + k0;
            if (vec && k0 + 8 <= job.K) {
                const f32x4 lo = *reinterpret_cast<const f32x4*>(p), hi = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) { v[i] = lo[i]; v[4 + i] = hi[i]; }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = k0 + i < job.K ? p[i] : 0.f;
            }
            store_pack(dst, job.rows, k0 >> 3, n, v);
        }
    }
}

size_t split_pack_elems(int64_t rows, int64_t K) { return (size_t)(ceil_div(K, GS_K) * 48 * rows); }

void launch_split_pack(hipStream_t s, SplitPackTable tab, bool kmajor, const float* src, uint16_t* dst) {
    int64_t blocks = 0;
    for (int i = 0; i < tab.n; ++i) {
        SplitPackJob& j = tab.j[i];
        j.blocks = (int)(kmajor ? ceil_div(j.rows, 256) * ceil_div(j.K, GS_K) : ceil_div(j.rows, 64) * ceil_div(j.K, 64));
        blocks += j.blocks;
    }
    if (blocks == 0) return;
    if (kmajor) hipLaunchKernelGGL(split_pack_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, tab, src, dst);
    else hipLaunchKernelGGL(split_pack_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, tab, src, dst);
}

// ---- products --------------------------------------------------------------------------------------------------------

// Workgroup = 64 WMB x 64 WNB tile of C, four waves as 2 x 2, each WMB x WNB blocks of v_mfma_f32_32x32x16_bf16.  K advances 16
// at a time through GS_STAGES LDS buffers that global_load_lds fills, as in gemm_direct_kernel, with its layout of A: row-major
// [row][16 k], 16-byte piece c of a row at place c ^ ((row / 4) % 4) (the lane's eight k are pieces 2g and 2g + 1); k-major
// [k][row], blocks of 16 rows of line k at block ^ ((k / 4) % 4).  Rows past the end are clamped, pieces of A past the end of K zeroed.
template <bool AK, int WMB, int WNB, int GS_STAGES>
__global__ __launch_bounds__(256, 2) void gemm_split_kernel(GemmDesc d) {
    constexpr int TM = 64 * WMB, TN = 64 * WNB;
    constexpr int LA = TM / 64, LB = (6 * WNB + 3) / 4;       // load instructions per wave and step
    constexpr int STAGE = TM * 4 + TN * 6;                    // 16-byte pieces
    extern __shared__ f32x4 gs_lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, g = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    int tile_x, tile_y, zz;
    gemm_tile_order(tile_x, tile_y, zz);
    const int m0 = tile_y * TM, n0 = tile_x * TN;
    const int split = zz % d.splits, z = zz / d.splits;
    const int k_begin = split * d.k_chunk;
    const int k_end = min(d.K, k_begin + d.k_chunk);
    const int steps = (k_end - k_begin + GS_K - 1) / GS_K;
    const bool tail = ((k_end - k_begin) % GS_K) != 0;        // the last step is not a whole one
    const int seg0 = d.k_seg ? k_begin / d.k_seg : 0;
    const int k_in_seg = d.k_seg ? k_begin - seg0 * d.k_seg : k_begin;
    const int64_t adv_a = AK ? (int64_t)GS_K * d.lda : GS_K, adv_b = (int64_t)48 * d.N;

    // slot v of a stage of A: the piece of the matrix that belongs there
    auto a_slot = [&](int v, int& row, int& k) {
        if (AK) {
            k = v / (TM / 4);
            row = 4 * ((v % (TM / 4)) ^ (4 * ((k >> 2) & 3)));
        } else {
            row = v >> 2;
            k = 4 * ((v & 3) ^ ((row >> 2) & 3));
        }
    };
    uint32_t offa[LA], offb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        int row, k;
        a_slot((4 * i + wave) * 64 + lane, row, k);
        offa[i] = AK ? (uint32_t)(k * d.lda + min(row, ((d.M - 1) & ~3) - m0)) : (uint32_t)(min(row, d.M - 1 - m0) * d.lda + k);
    }
    // 64 rows of one of the six (plane, half) pairs per instruction; where four waves do not divide them some are loaded twice
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int v = min(4 * i + wave, 6 * WNB - 1);
        offb[i] = (uint32_t)((v / WNB) * d.N + min(n0 + (v % WNB) * 64 + lane, d.N - 1)) * 8u;
    }
    auto load16 = [&](const void* src, int slot) {
        __builtin_amdgcn_global_load_lds((gs_global_ptr*)src, (gs_lds_ptr*)(gs_lds + slot), 16, 0, 0);
    };
    // the lane's eight values of k of row r of block t of A
    const int ra = (wm * 32 * WMB + r) * 4 + ((2 * g) ^ ((r >> 2) & 3));
    auto read_a = [&](int base, int t, f32x4& lo, f32x4& hi) {
        if constexpr (AK) {
            const float* as = reinterpret_cast<const float*>(gs_lds + base);
            const int b16 = 2 * (wm * WMB + t) + (r >> 4);
            const float* p0 = as + 8 * g * TM + 16 * (b16 ^ (2 * g)) + (r & 15);
            const float* p1 = as + (8 * g + 4) * TM + 16 * (b16 ^ (2 * g + 1)) + (r & 15);
#pragma unroll
            for (int j = 0; j < 4; ++j) { lo[j] = p0[j * TM]; hi[j] = p1[j * TM]; }
        } else {
            lo = gs_lds[base + ra + 128 * t];
            hi = gs_lds[base + (ra ^ 1) + 128 * t];
        }
    };
    const int rb = TM * 4 + g * TN + wn * 32 * WNB + r;
    auto read_b = [&](int base, int t, int plane) { return gs_lds[base + rb + 2 * plane * TN + 32 * t]; };

    f32x16 acc[WMB][WNB], small[WMB][WNB], sum[AK ? WMB : 1][AK ? WNB : 1];
    // The whole contraction: PLAIN by fp32 matrix instructions
    auto contract = [&](auto plain_t) __attribute__((always_inline)) {
        constexpr bool PLAIN = decltype(plain_t)::value;
        int seg_left = d.k_seg ? d.k_seg - k_in_seg : INT_MAX;
        const float* A = d.A + z * d.sa1 + seg0 * d.sa_seg + (AK ? (int64_t)k_in_seg * d.lda + m0 : (int64_t)m0 * d.lda + k_in_seg);
        const uint16_t* B = d.Bs + z * d.sb1 + (int64_t)(k_begin / GS_K) * adv_b;
        // request of step `step` (they come in order) into buffer `buf`
        auto request = [&](int step, int buf) {
            const int base = buf * STAGE;
#pragma unroll
            for (int i = 0; i < LB; ++i) load16(B + offb[i], base + TM * 4 + min(4 * i + wave, 6 * WNB - 1) * 64);
            B += adv_b;
            if (tail && step == steps - 1) {
                const int left = k_end - k_begin - step * GS_K;   // 1 .. 15
#pragma unroll
                for (int i = 0; i < LA; ++i) {
                    int row, k;
                    const int v = (4 * i + wave) * 64 + lane;
                    a_slot(v, row, k);
                    if (k < left) load16(A + offa[i], base + (4 * i + wave) * 64);
                    else gs_lds[base + v] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < LA; ++i) load16(A + offa[i], base + (4 * i + wave) * 64);
            A += adv_a;
            seg_left -= GS_K;
            if (seg_left == 0) {
                seg_left = d.k_seg;
                A += d.sa_seg - (AK ? (int64_t)d.k_seg * d.lda : (int64_t)d.k_seg);
            }
        };
#pragma unroll
        for (int i = 0; i < WMB; ++i)
#pragma unroll
            for (int j = 0; j < WNB; ++j) {
                acc[i][j] = small[i][j] = f32x16{};
                if constexpr (AK) sum[i][j] = f32x16{};
            }
        auto end_run = [&](int done) {
            if constexpr (AK) {
                if (done % GT_RUN == 0) {
                    asm volatile("" ::: "memory");   // a branch, not a selection of every sum in every step
#pragma unroll
                    for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
                        for (int nt = 0; nt < WNB; ++nt) {
                            sum[mt][nt] += acc[mt][nt];
                            acc[mt][nt] = f32x16{};
                        }
                }
            }
        };
        // The loads of step i are in and everybody's reads of step i - 1 are done.  While a later step is still to be requested the
        // GS_STAGES - 2 youngest steps may stay in flight: the last step, whose count of loads may be another, is not among them.
        auto wait = [&](int i) {
            if (i + GS_STAGES - 1 < steps) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((GS_STAGES - 2) * (LA + LB)) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        int buf = 0;
        auto advance = [&](int i) {   // to step i, whose request GS_STAGES - 1 steps ahead goes into the buffer just left
            wait(i);
            if (i + GS_STAGES - 1 < steps) request(i + GS_STAGES - 1, buf == 0 ? GS_STAGES - 1 : buf - 1);
        };
#pragma unroll
        for (int i = 0; i < GS_STAGES - 1; ++i)
            if (i < steps) request(i, i);
        if constexpr (PLAIN) {
            for (int i = 0; i < steps; ++i) {
                advance(i);
                const int base = buf * STAGE;
#pragma unroll
                for (int nt = 0; nt < WNB; ++nt) {
                    const u32x4 bh = __builtin_bit_cast(u32x4, read_b(base, nt, 0)), bm = __builtin_bit_cast(u32x4, read_b(base, nt, 1)),
                                bl = __builtin_bit_cast(u32x4, read_b(base, nt, 2));
                    float b[8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        b[2 * j] = (__uint_as_float(bl[j] << 16) + __uint_as_float(bm[j] << 16)) + __uint_as_float(bh[j] << 16);
                        b[2 * j + 1] = (__uint_as_float(bl[j] & 0xffff0000u) + __uint_as_float(bm[j] & 0xffff0000u)) + __uint_as_float(bh[j] & 0xffff0000u);
                    }
#pragma unroll
                    for (int mt = 0; mt < WMB; ++mt) {
                        f32x4 lo, hi;
                        read_a(base, mt, lo, hi);
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j], j < 4 ? lo[j & 3] : hi[j & 3], acc[mt][nt], 0, 0, 0);
                    }
                }
                buf = buf + 1 == GS_STAGES ? 0 : buf + 1;
                end_run(i + 1);
            }
        } else {
            for (int i = 0; i < steps; ++i) {
                advance(i);
                const int base = buf * STAGE;
                bf16x8 b[WNB][3];
#pragma unroll
                for (int t = 0; t < WNB; ++t)
#pragma unroll
                    for (int p = 0; p < 3; ++p) b[t][p] = __builtin_bit_cast(bf16x8, read_b(base, t, p));
#pragma unroll
                for (int mt = 0; mt < WMB; ++mt) {
                    f32x4 lo, hi;
                    read_a(base, mt, lo, hi);
                    const Split8 a = split8(lo, hi);
#define GS_MM(P, Y, C)                                   \
    _Pragma("unroll") for (int nt = 0; nt < WNB; ++nt) C[mt][nt] = \
        __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[nt][P], bf16x8_of(a.Y), C[mt][nt], 0, 0, 0)
                    GS_MM(2, h, small);
                    GS_MM(0, h, acc);
                    GS_MM(1, h, small);
                    GS_MM(1, m, small);
                    GS_MM(0, m, small);
                    GS_MM(0, l, small);
#undef GS_MM
                }
                buf = buf + 1 == GS_STAGES ? 0 : buf + 1;
                end_run(i + 1);
            }
        }
#pragma unroll
        for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
            for (int nt = 0; nt < WNB; ++nt) {
                if constexpr (!PLAIN) acc[mt][nt] += small[mt][nt];
                if constexpr (AK) acc[mt][nt] += sum[mt][nt];
            }
    };
    contract(std::false_type{});
    // lane (r, g) holds acc[mt][nt][4q + i] = C[.. + r][.. + 8q + 4g + i] of every 32 x 32 block
    bool again = false;
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt)
#pragma unroll
        for (int nt = 0; nt < WNB; ++nt)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (m0 + (wm * WMB + mt) * 32 + r < d.M && n0 + (wn * WNB + nt) * 32 + 8 * q + 4 * g < d.N)
#pragma unroll
                    for (int i = 0; i < 4; ++i) again |= !(fabsf(acc[mt][nt][4 * q + i]) < INFINITY);
    if (__syncthreads_or(again)) contract(std::true_type{});

    const bool plain = d.splits > 1;   // partial sums go out as they are; the reduction applies the epilogue
    float* C = plain ? d.part + ((int64_t)z * d.splits + split) * d.part_stride : d.C ? d.C + z * d.sc1 : nullptr;
    const int ldc = plain ? d.N : d.ldc;
    const float* R = (plain || !d.R) ? nullptr : d.R + z * d.sc1;
    const float* bias = (plain || !d.bias) ? nullptr : d.bias + z * d.sbias1;
    const bool vec = plain ? (d.N & 3) == 0 : d.c_vec != 0;
#pragma unroll
    for (int mt = 0; mt < WMB; ++mt) {
        const int m = m0 + (wm * WMB + mt) * 32 + r;
        if (m >= d.M) continue;
#pragma unroll
        for (int nt = 0; nt < WNB; ++nt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + (wn * WNB + nt) * 32 + 8 * q + 4 * g;
                if (n >= d.N) continue;
                const int64_t at = (int64_t)m * ldc + n;
                f32x4 v = f32x4{acc[mt][nt][4 * q], acc[mt][nt][4 * q + 1], acc[mt][nt][4 * q + 2], acc[mt][nt][4 * q + 3]};
                if (vec && n + 3 < d.N) {
                    if (!plain) {
                        v *= d.alpha;
                        if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
                        if (R) v += *reinterpret_cast<const f32x4*>(R + at);
                        if (d.G) {
                            f32x4 u;
#pragma unroll
                            for (int i = 0; i < 4; ++i) u[i] = gelu_f32(v[i]);
                            *reinterpret_cast<f32x4*>(d.G + at) = u;
                        }
                    }
                    if (C) *reinterpret_cast<f32x4*>(C + at) = v;
                } else {
                    for (int i = 0; i < 4 && n + i < d.N; ++i) {
                        float u = v[i];
                        if (!plain) {
                            u *= d.alpha;
                            if (bias) u += bias[n + i];
                            if (R) u += R[at + i];
                            if (d.G) d.G[at + i] = gelu_f32(u);
                        }
                        if (C) C[at + i] = u;
                    }
                }
            }
    }
}

// Tile and split of a product: the pair with the smallest estimate of (K steps + six for the first loads and the epilogue) x
// (workgroups of the busiest compute unit) x (time of a step) + the pass that adds the partial sums.  Times of a step in us,
// measured on 3100 tokens x 512 x 512 to 2048 and on weight gradients of 2048 x 512: alone on its compute unit a workgroup, whose four
// waves read, split and multiply one after the other, takes longer than beside others.  (3100 x 512 x 2048: 128 x 128 in four parts
// 50.5 us, 64 x 128 in two 50.5, 64 x 64 60.7, 64 x 128 62.7, 128 x 128 87.6; the fp32 instruction, 64 x 128, 75.)
struct GsPlan {
    int wmb, wnb, splits;
};
static GsPlan gs_plan(int64_t M, int64_t N, int64_t K, int batch, int max_splits, bool ak) {
    static const struct { int wmb, wnb; double alone[2], beside[2]; } tiles[3] = {
        {2, 2, {0.65, 0.735}, {0.56, 0.58}}, {1, 2, {0.47, 0.49}, {0.31, 0.35}}, {1, 1, {0.36, 0.40}, {0.235, 0.285}}};
    GsPlan best{2, 2, 1};
    double best_us = 1e30;
    for (const auto& t : tiles)
        for (int sp = 1; sp <= max_splits; ++sp) {
            if (sp > 1 && K / sp < 16 * GS_K) break;
            const double wgs = (double)ceil_div(M, 64 * t.wmb) * (double)ceil_div(N, 64 * t.wnb) * batch * sp;
            const double steps = (double)ceil_div(ceil_div(K, sp), GS_K) + 6.0;
            double us = wgs <= 256.0 ? steps * t.alone[ak] : ceil(wgs / 256.0) * steps * t.beside[ak];
            if (sp > 1) us += 3.0 + (sp + 1.0) * (double)M * (double)N * batch * 4.0 / 4.0e6;
            if (us < best_us) {
                best_us = us;
                best = GsPlan{t.wmb, t.wnb, sp};
            }
        }
    return best;
}

bool gemm_split_takes(const float* A, int lda, int64_t sa1, int64_t sa_seg, bool a_kmajor, int K, int k_seg) {
    return (reinterpret_cast<uintptr_t>(A) & 15) == 0 && lda % 4 == 0 && sa1 % 4 == 0 && sa_seg % 4 == 0 && (a_kmajor || K % 4 == 0) &&
           k_seg % GS_K == 0 && (int64_t)128 * lda < (int64_t(1) << 29);
}

int launch_gemm_split(hipStream_t s, GemmDesc d) {
    if (d.splits < 1) d.splits = 1;
    if (d.batch < 1) d.batch = 1;
    if (!gemm_split_takes(d.A, d.lda, d.sa1, d.sa_seg, d.a_kmajor != 0, d.K, d.k_seg) || d.inner > 1 || (int64_t)6 * d.N * 8 >= (int64_t(1) << 31) || d.sb1 % 8 != 0)
        return BLS_EUNSUPPORTED;
    auto aligned = [](const float* p, int ld, int64_t s1) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 4 == 0 && s1 % 4 == 0; };
    d.c_vec = aligned(d.C, d.ldc, d.sc1) && aligned(d.R, 0, 0) && aligned(d.bias, 0, d.sbias1) && aligned(d.G, 0, 0) ? 1 : 0;
    const GsPlan p = gs_plan(d.M, d.N, d.K, d.batch, d.splits, d.a_kmajor != 0);
    d.k_chunk = (int)ceil_div(ceil_div(d.K, p.splits), GS_K) * GS_K;
    d.splits = (int)ceil_div(d.K, d.k_chunk);
    d.part_stride = (int64_t)d.M * d.N;
    const dim3 grid((unsigned)ceil_div(d.N, 64 * p.wnb), (unsigned)ceil_div(d.M, 64 * p.wmb), d.batch * d.splits);
#define GS_LAUNCH(AK, WMB, WNB, ST) \
    hipLaunchKernelGGL((gemm_split_kernel<AK, WMB, WNB, ST>), grid, dim3(256), ST * 16 * (64 * 4 * WMB + 64 * 6 * WNB), s, d)
#define GS_TILE(AK)                                 \
    do {                                            \
        if (p.wmb == 2) GS_LAUNCH(AK, 2, 2, 3);     \
        else if (p.wnb == 2) GS_LAUNCH(AK, 1, 2, 3); \
        else GS_LAUNCH(AK, 1, 1, 4);                \
    } while (0)
    if (d.a_kmajor) GS_TILE(true);
    else GS_TILE(false);
#undef GS_TILE
#undef GS_LAUNCH
    if (d.splits > 1)
        launch_split_reduce(s, d.part, d.splits, d.M, d.N, d.batch, d.alpha, d.bias, d.sbias1, d.R, d.ldc, d.C, d.sc1, d.c_vec != 0);
    return BLS_OK;
}
