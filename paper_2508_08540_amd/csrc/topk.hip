// Deterministic loss-based top-k selection (Section 4.2): the k highest-loss samples in rank order.
//
// Every loss is mapped to a 64-bit sort word whose unsigned order is the selection order:
//   high 32 bits: the float's bits made monotone (sign flip), with -0 folded into +0 and every
//                 NaN folded into the largest word, so NaN ranks above +inf;
//   low 32 bits:  ~index, so that among equal losses the smaller index is the larger word.
// All words are distinct, hence exactly one result is correct and no stability argument is needed.
//
// Pools of up to TOPK_RANK_MAX samples are ranked by counting in one launch; pools of up to TOPK_SORT_MAX are sorted whole by
// four radix passes of one launch each; larger ones take radix-select of the k-th word, ordered compaction of the selected
// words, and an LSD radix sort of those k words.
#include <mutex>

#include "common.h"

// Ranking by counting needs no scratch and costs 24.6 us at 16384 (four sorting passes: 22 us at 16385); sorting a pool of
// 2^19 whole takes 73 us for any k, selecting first 98 (k = N / 50) to 120 us (k = N); at 2^20 about 117 against 86 to 105 us.
#define TOPK_RANK_MAX 16384

__device__ __forceinline__ uint32_t loss_key(float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0xffffffffu;  // NaN: above +inf
    if (u == 0x80000000u) u = 0u;                              // -0 == +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint32_t job_key(const SelJob& job, int i) {
    const float v = job.losses[i];
    return loss_key(v < job.floor ? job.floor : v);   // a NaN stays one
}

// Rank by counting: the rank of a sample is the number of samples that precede it, so each workgroup ranks 64 samples (one per
// lane) against the whole pool, which its 16 waves walk in chunks of 64 keys from LDS (every lane reads the same four keys per
// 16-byte read).  Chunks left of the workgroup's own count equal keys, chunks right of it do not: the tie rule costs nothing
// but in the one chunk where both orders occur.  Bound: vector instructions, two per pair of samples; N^2 of them still beat
// the N log^2 N of a bitonic network with its 100 barriers in one workgroup because all compute units take part.
// N = 512 / 4096 / 16384: 9.8 -> 4.3, 38 -> 8.7, 157 -> 24.5 us against the bitonic network.
__global__ __launch_bounds__(1024) void topk_rank_kernel(SelJobs jobs, int N) {
    const SelJob& job = jobs.j[blockIdx.y];
    const float* __restrict__ losses = job.losses;
    extern __shared__ __align__(16) uint32_t rank_lds[];   // the keys, then [16][64] partial ranks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_chunks = (N + 63) >> 6, own = blockIdx.x;
    for (int i = tid; i < n_chunks * 64; i += 1024) rank_lds[i] = i < N ? job_key(job, i) : 0u;   // no loss has key 0
    __syncthreads();
    const uint32_t mine = rank_lds[own * 64 + lane];
    uint32_t before = 0;
    for (int c = wave; c < n_chunks; c += 16) {
        const uint4* q = reinterpret_cast<const uint4*>(rank_lds + c * 64);
        if (c < own) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint4 v = q[j];
                before += (v.x >= mine) + (v.y >= mine) + (v.z >= mine) + (v.w >= mine);
            }
        } else if (c > own) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint4 v = q[j];
                before += (v.x > mine) + (v.y > mine) + (v.z > mine) + (v.w > mine);
            }
        } else {
            for (int j = 0; j < 64; ++j) {
                const uint32_t v = rank_lds[c * 64 + j];
                before += v > mine || (v == mine && j < lane);
            }
        }
    }
    __syncthreads();   // the partial ranks overwrite the keys
    rank_lds[tid] = before;
    __syncthreads();
    if (wave == 0) {
        uint32_t rank = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) rank += rank_lds[w * 64 + lane];
        const int i = own * 64 + lane;
        if (job.chosen && i < N) job.chosen[i] = rank < (uint32_t)job.k;
        if (i < N && rank < (uint32_t)job.k) {
            job.idx_out[rank] = i;
            if (job.val_out) job.val_out[rank] = losses[i];
        }
    }
}

// Inverse of loss_key for every key that determines the float uniquely; NaN keys and the zero key
// (shared by +0 and -0) do not, those values are fetched from the loss array.
__device__ __forceinline__ bool key_to_loss(uint32_t key, float* v) {
    if (key == 0xffffffffu || key == 0x80000000u) return false;
    uint32_t u = (key & 0x80000000u) ? (key & 0x7fffffffu) : ~key;
    *v = __uint_as_float(u);
    return true;
}

// ---- medium pools: the whole pool in four radix passes ----------------------------------------------------------------
//
// These pools are bound by launches, not by bytes (50 000 losses are 200 KB): selecting first, and scanning a digit table
// between the passes, took 21 launches of 2 to 6 us each.  Here the pool is sorted whole in five launches.  The pool is at most
// SORT_TILES tiles of RITER x 1024 elements, so the digit table [tile][256] is small enough that every workgroup adds up its
// columns itself (tiles before its own, and all of them) instead of waiting for a scan, and the pass that places an element
// also counts it in the table of the next pass: the destination tile and the next digit are known at that point.  These counts
// meet in LDS first (16 bits each, a tile has at most 8192 elements), since all elements of a run may share the next digit.
// k = N, N = 50 000 / 131 072 / 524 288: 79 -> 29, 95 -> 40, 120 -> 73 us (with the table's loads one after another: 37, 51,
// 85).  What is left is five launches, each a chain of load, table sum, ranking rounds and scattered stores.

#define SORT_TILES 64   // 64 tiles of 8 x 1024 elements hold TOPK_SORT_MAX
#define SORT_TABLE (SORT_TILES * 256)

// Tile of a workgroup.  Workgroups are dealt to the eight XCDs in turn; an XCD takes consecutive tiles, so that the short runs its
// tiles write per digit lie side by side: a cache line that several XCDs write leaves each one's L2 by itself.
__device__ __forceinline__ int sort_tile() {
    const int tiles = gridDim.x, r = blockIdx.x & 7, per = tiles >> 3, rem = tiles & 7;
    return r * per + min(r, rem) + ((int)blockIdx.x >> 3);
}

// Digit counts of the first pass; clears the tables of the other three.
template <int RITER>
__global__ __launch_bounds__(1024) void sort_count_kernel(SelJobs jobs, int N) {
    const SelJob& job = jobs.j[blockIdx.y];
    uint32_t* __restrict__ tables = job.tables;
    __shared__ uint32_t cnt[256];
    const int tid = threadIdx.x, tile = sort_tile();
    const int base = tile * (RITER * 1024);
    // requested before anything else, past the end the last one again: no branch that would wait for its load
    uint32_t key[RITER];
#pragma unroll
    for (int it = 0; it < RITER; ++it) key[it] = ~job_key(job, min(base + it * 1024 + tid, N - 1));
    if (tid < 256) cnt[tid] = 0u;
    else tables[(size_t)(tid >> 8) * SORT_TABLE + tile * 256 + (tid & 255)] = 0u;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RITER; ++it)
        if (base + it * 1024 + tid < N) atomicAdd(&cnt[key[it] & 255u], 1u);
    __syncthreads();
    if (tid < 256) tables[tile * 256 + tid] = cnt[tid];
}

// One stable pass over the sort keys ~loss_key (ascending order is rank order).  A wave ranks its RITER x 64 consecutive
// elements in rounds of 64 by ballots, counting each digit as it goes; the four groups of 256 threads add up a quarter of the
// table each.  PASS 0 reads the losses, PASS 3 stores the first k of the result.
template <int RITER, int PASS>
__global__ __launch_bounds__(1024) void sort_pass_kernel(SelJobs jobs, int N) {
    const SelJob& job = jobs.j[blockIdx.y];
    const uint2* __restrict__ in = PASS == 2 ? job.b : job.a;
    uint2* __restrict__ out = PASS == 1 ? job.b : job.a;
    const uint32_t* __restrict__ table = job.tables + PASS * SORT_TABLE;
    uint32_t* __restrict__ table_next = job.tables + (PASS + 1) * SORT_TABLE;
    constexpr int RTILE = RITER * 1024, SHIFT = 8 * PASS;
    __shared__ uint32_t cnt[16][256];
    __shared__ uint32_t part[2][4][256];
    __shared__ uint32_t wave_total[4];
    __shared__ uint32_t next[PASS < 3 ? SORT_TABLE / 2 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tiles = gridDim.x, tile = sort_tile();
    const int wbase = tile * RTILE + wave * (RITER * 64);
    uint32_t key[RITER], id[RITER];
#pragma unroll
    for (int it = 0; it < RITER; ++it) {
        // past the end the last one again, which is not ranked: no branch that would wait for its load before the table's
        const int i = wbase + it * 64 + lane, at = min(i, N - 1);
        if (PASS == 0) {
            key[it] = ~job_key(job, at);
            id[it] = (uint32_t)i;
        } else {
            const uint2 v = in[at];
            key[it] = v.x;
            id[it] = v.y;
        }
    }
    {
        const int d = tid & 255, g = tid >> 8;
        uint32_t v[SORT_TILES / 4], all = 0, left = 0;
#pragma unroll
        for (int j = 0; j < SORT_TILES / 4; ++j) v[j] = g + 4 * j < tiles ? table[(g + 4 * j) * 256 + d] : 0u;   // all in flight together
#pragma unroll
        for (int j = 0; j < SORT_TILES / 4; ++j) {
            all += v[j];
            left += g + 4 * j < tile ? v[j] : 0u;
        }
        part[0][g][d] = all;
        part[1][g][d] = left;
    }
    for (int i = tid; i < 16 * 256; i += 1024) cnt[i >> 8][i & 255] = 0u;
    if (PASS < 3)
        for (int i = tid; i < tiles * 128; i += 1024) next[i] = 0u;
    __syncthreads();
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t rank[RITER];
#pragma unroll
    for (int it = 0; it < RITER; ++it) {
        const bool valid = wbase + it * 64 + lane < N;
        const uint32_t d = (key[it] >> SHIFT) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t v = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? v : ~v;
        }
        rank[it] = cnt[wave][d] + (uint32_t)__popcll(peers & lt);
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & lt) == 0ull) cnt[wave][d] += (uint32_t)__popcll(peers);   // lowest peer advances the count
        __builtin_amdgcn_wave_barrier();
    }
    // thread d < 256: first output slot of digit d = elements of smaller digits + those of d in tiles before this one
    uint32_t total = 0, incl = 0;
    if (tid < 256) {
        total = (part[0][0][tid] + part[0][1][tid]) + (part[0][2][tid] + part[0][3][tid]);
        incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t below = __shfl_up(incl, o, 64);
            if (lane >= o) incl += below;
        }
        if (lane == 63) wave_total[wave] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t run = incl - total + (part[1][0][tid] + part[1][1][tid]) + (part[1][2][tid] + part[1][3][tid]);
        for (int w = 0; w < wave; ++w) run += wave_total[w];
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t c = cnt[w][tid];
            cnt[w][tid] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RITER; ++it) {
        if (wbase + it * 64 + lane >= N) continue;
        const uint32_t pos = cnt[wave][(key[it] >> SHIFT) & 255u] + rank[it];
        if (PASS < 3) {
            out[pos] = make_uint2(key[it], id[it]);
            const uint32_t slot = (pos / RTILE) * 256u + ((key[it] >> (SHIFT + 8)) & 255u);
            atomicAdd(&next[slot >> 1], (slot & 1u) ? 65536u : 1u);
            continue;
        }
        if (job.chosen) job.chosen[id[it]] = pos < (uint32_t)job.k;
        if (pos < (uint32_t)job.k) {
            job.idx_out[pos] = (int32_t)id[it];
            if (job.val_out) {
                float v;
                if (!key_to_loss(~key[it], &v)) v = job.losses[id[it]];
                job.val_out[pos] = v;
            }
        }
    }
    if (PASS == 3) return;
    __syncthreads();
    for (int i = tid; i < tiles * 128; i += 1024) {
        const uint32_t v = next[i];
        if (v & 65535u) atomicAdd(&table_next[2 * i], v & 65535u);
        if (v >> 16) atomicAdd(&table_next[2 * i + 1], v >> 16);
    }
}

static void carve_sort(Carver& c, int64_t N, SelJob& job) {
    job.tables = c.take<uint32_t>(4 * SORT_TABLE);
    job.a = c.take<uint2>(N);
    job.b = c.take<uint2>(N);
}

template <int RITER>
static void launch_sort(hipStream_t s, const SelJobs& jobs, int n_jobs, int N) {
    const dim3 grid((unsigned)((N + RITER * 1024 - 1) / (RITER * 1024)), n_jobs), block(1024);
    hipLaunchKernelGGL(sort_count_kernel<RITER>, grid, block, 0, s, jobs, N);
    hipLaunchKernelGGL((sort_pass_kernel<RITER, 0>), grid, block, 0, s, jobs, N);
    hipLaunchKernelGGL((sort_pass_kernel<RITER, 1>), grid, block, 0, s, jobs, N);
    hipLaunchKernelGGL((sort_pass_kernel<RITER, 2>), grid, block, 0, s, jobs, N);
    hipLaunchKernelGGL((sort_pass_kernel<RITER, 3>), grid, block, 0, s, jobs, N);
}

// TOPK_RANK_MAX < N <= TOPK_SORT_MAX; `scratch_base` as below, n_jobs times.  The fewest rounds that keep the pool within
// SORT_TILES tiles.
static int launch_topk_medium(bls_ctx* ctx, char* scratch_base, SelJobs jobs, int n_jobs, int64_t N) {
    Carver c(scratch_base);
    for (int i = 0; i < n_jobs; ++i) carve_sort(c, N, jobs.j[i]);
    if (N <= 1 * 65536) launch_sort<1>(ctx->stream, jobs, n_jobs, (int)N);
    else if (N <= 2 * 65536) launch_sort<2>(ctx->stream, jobs, n_jobs, (int)N);
    else if (N <= 4 * 65536) launch_sort<4>(ctx->stream, jobs, n_jobs, (int)N);
    else launch_sort<8>(ctx->stream, jobs, n_jobs, (int)N);
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}

// ---- large pools ----------------------------------------------------------------------------------
//
// 1. Two-level radix select of the k-th largest key: a 2048-bin histogram of the top 11 key bits gives the bin b1 that
//    holds it, a second histogram of the next 11 bits over the members of b1 gives the 22-bit prefix `thr`: the M
//    elements with key >> 10 >= thr are selected (M >= k; the excess is at most the members of one 22-bit prefix).
//    Histograms are aggregated per wave before they touch LDS (losses crowd into a few exponent bins).
// 2. The selected elements are compacted, in index order, into (sort key, index) pairs; the sort key is hi - key
//    (hi bounds every key), so that ascending order is rank order and the keys only span the range that occurs.
// 3. Stable LSD radix sort of the M pairs, 8 bits per pass, with as many passes as that range needs (the later passes
//    exit at once).  Stability keeps equal losses in ascending index order, which is the tie rule.
// 4. The first k pairs are the result: the last pass stores indices and losses instead of pairs.
// Nothing is read back to the host: grids are sized for the worst case M == N and blocks past M exit.

#define SEL_BINS 2048
#define TILE 2048          // elements per 256-thread block: 8 consecutive elements per thread
#define SCAN_CHUNK 2048
// Radix passes: a block of 256 threads handles RITER * 256 elements (each wave ranks RITER * 64 of them in
// rounds of 64); 8 rounds for pools below 2^22, 16 for very large ones (longer runs per digit when scattering).

struct SelInfo {
    uint32_t bin;        // b1
    uint32_t above;      // elements in bins above b1
    uint32_t thr;        // selected: key >> 10 >= thr
    uint32_t M;          // number of selected elements
    uint32_t hi;         // no key is larger; sort key = hi - key
    uint32_t n_passes;   // 8-bit passes that cover hi - (thr << 10)
};

__global__ __launch_bounds__(256) void zero_u32_kernel(uint32_t* p, int64_t n) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0u;
}

// Elements 4 q .. 4 q + 3 (zero key, invalid, past N); VEC: the array allows 16-byte loads.
template <bool VEC>
__device__ __forceinline__ void load_keys4(const float* __restrict__ losses, int64_t N, int64_t q, uint32_t (&key)[4], bool (&ok)[4]) {
    const int64_t i0 = q * 4;
    if (VEC && i0 + 3 < N) {
        const float4 v = *reinterpret_cast<const float4*>(losses + i0);
        key[0] = loss_key(v.x); key[1] = loss_key(v.y); key[2] = loss_key(v.z); key[3] = loss_key(v.w);
        ok[0] = ok[1] = ok[2] = ok[3] = true;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ok[j] = i0 + j < N;
            key[j] = ok[j] ? loss_key(losses[i0 + j]) : 0u;
        }
    }
}

// LEVEL 1: bins of key >> 21 over all elements.  Losses crowd into a handful of exponent bins, so every bin has
// SUB counters in LDS and a lane adds to counter lane % SUB: the lanes of a wave that meet in one bin spread over SUB
// addresses.  LEVEL 2: bins of (key >> 10) & 2047 over the members of info->bin only (those bits are spread evenly).
// 1024 threads per histogram: the loop waits for memory (256 threads, two to eight workgroups per unit: 25 + 29 us at 2^24
// keys, now 15 + 19), while every further histogram costs a clear and a fold of 2048 bins.
#define HIST_THREADS 1024
template <int LEVEL, bool VEC>
__global__ __launch_bounds__(HIST_THREADS) void sel_hist_kernel(const float* __restrict__ losses, int64_t N, const SelInfo* __restrict__ info,
                                                       uint32_t* __restrict__ hist) {
    constexpr int SUB = LEVEL == 1 ? 8 : 1;
    __shared__ uint32_t h[SEL_BINS * SUB];
    for (int i = threadIdx.x; i < SEL_BINS * SUB; i += HIST_THREADS) h[i] = 0u;
    __syncthreads();
    const uint32_t b1 = LEVEL == 2 ? info->bin : 0u;
    const uint32_t sub = threadIdx.x & (SUB - 1);
    const int64_t quads = (N + 3) >> 2, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < quads; q += 2 * stride) {
        uint32_t key[2][4];
        bool ok[2][4] = {{false, false, false, false}, {false, false, false, false}};
        load_keys4<VEC>(losses, N, q, key[0], ok[0]);
        if (q + stride < quads) load_keys4<VEC>(losses, N, q + stride, key[1], ok[1]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (LEVEL == 1) {
                    if (ok[u][j]) atomicAdd(&h[(key[u][j] >> 21) * SUB + sub], 1u);
                } else {
                    if (ok[u][j] && (key[u][j] >> 21) == b1) atomicAdd(&h[(key[u][j] >> 10) & (SEL_BINS - 1)], 1u);
                }
            }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SEL_BINS; i += HIST_THREADS) {
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < SUB; ++u) c += h[i * SUB + u];
        if (c) atomicAdd(&hist[i], c);
    }
}

// One block: suffix counts over the bins; the bin sought is the largest one whose suffix count reaches `want`.
// LEVEL 1: want = k; stores bin, above and hi.  LEVEL 2: want = k - above over the sub-bins of b1; stores thr, M, n_passes.
template <int LEVEL>
__global__ __launch_bounds__(256) void sel_threshold_kernel(const uint32_t* __restrict__ hist, uint32_t k, SelInfo* __restrict__ info) {
    __shared__ uint32_t part[256];
    __shared__ uint32_t top_bin;
    const uint32_t want = LEVEL == 1 ? k : k - info->above;
    uint32_t mine[8], tot = 0;
    if (threadIdx.x == 0) top_bin = 0u;
    for (int j = 0; j < 8; ++j) {
        mine[j] = hist[threadIdx.x * 8 + j];
        tot += mine[j];
    }
    part[threadIdx.x] = tot;
    __syncthreads();
    if (LEVEL == 1)
        for (int j = 0; j < 8; ++j)
            if (mine[j]) atomicMax(&top_bin, threadIdx.x * 8 + j);
    // inclusive suffix sum over threads (thread t: bins 8t .. 8t+7)
    for (int o = 1; o < 256; o <<= 1) {
        uint32_t add = (threadIdx.x + o < 256) ? part[threadIdx.x + o] : 0u;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    uint32_t above = part[threadIdx.x] - tot;  // elements in bins of higher threads
    for (int j = 7; j >= 0; --j) {
        uint32_t with = above + mine[j];
        if (above < want && with >= want) {
            const uint32_t b = threadIdx.x * 8 + j;
            if (LEVEL == 1) {
                info->bin = b;
                info->above = above;
                info->hi = top_bin == SEL_BINS - 1 ? 0xffffffffu : ((top_bin + 1u) << 21) - 1u;
            } else {
                const uint32_t thr = (info->bin << 11) | b;
                const uint32_t range = info->hi - (thr << 10);   // sort keys lie in [0, range]
                info->thr = thr;
                info->M = info->above + with;
                info->n_passes = range < 256u ? 1u : (32u - (uint32_t)__clz(range) + 7u) / 8u;   // the last pass stores the result
            }
        }
        above = with;
    }
}

__device__ __forceinline__ uint32_t block_exclusive_scan_256(uint32_t v, uint32_t* total) {
    // inclusive scan inside each wave by shuffles, then the four wave totals through LDS
    __shared__ uint32_t wave_total[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t below = __shfl_up(incl, o, 64);
        if (lane >= o) incl += below;
    }
    if (lane == 63) wave_total[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += wave_total[w];
    const uint32_t all = (wave_total[0] + wave_total[1]) + (wave_total[2] + wave_total[3]);
    __syncthreads();   // wave_total may be written again by the next call
    if (total) *total = all;
    return before + incl - v;
}

// The 8 consecutive elements of a thread (two quads)
template <bool VEC>
__device__ __forceinline__ uint32_t load_tile_keys(const float* __restrict__ losses, int64_t N, uint32_t thr, uint32_t (&key)[8], bool (&sel)[8]) {
    const int64_t q0 = ((int64_t)blockIdx.x * TILE + threadIdx.x * 8) >> 2;
    uint32_t c = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t kq[4];
        bool ok[4];
        load_keys4<VEC>(losses, N, q0 + h, kq, ok);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            key[4 * h + j] = kq[j];
            sel[4 * h + j] = ok[j] && (kq[j] >> 10) >= thr;
            c += sel[4 * h + j] ? 1u : 0u;
        }
    }
    return c;
}

template <bool VEC>
__global__ __launch_bounds__(256) void sel_count_kernel(const float* __restrict__ losses, int64_t N, const SelInfo* __restrict__ info,
                                                        uint32_t* __restrict__ counts) {
    uint32_t key[8];
    bool sel[8];
    const uint32_t c = load_tile_keys<VEC>(losses, N, info->thr, key, sel);
    uint32_t total;
    block_exclusive_scan_256(c, &total);
    if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// counts has been exclusive-scanned into offsets.  The selected pairs of a tile are gathered in LDS and stored side by side: from
// the threads' own eight elements every store would go to 64 places (16 M keys, 4 M selected: 29 -> 19 us).
template <bool VEC>
__global__ __launch_bounds__(256) void sel_compact_kernel(const float* __restrict__ losses, int64_t N, const SelInfo* __restrict__ info,
                                                          const uint32_t* __restrict__ offsets, uint2* __restrict__ pairs) {
    __shared__ uint2 buf[TILE];
    const uint32_t hi = info->hi;
    const int64_t base = (int64_t)blockIdx.x * TILE + threadIdx.x * 8;
    uint32_t key[8];
    bool sel[8];
    const uint32_t c = load_tile_keys<VEC>(losses, N, info->thr, key, sel);
    uint32_t total, pos = block_exclusive_scan_256(c, &total);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (sel[j]) buf[pos++] = make_uint2(hi - key[j], (uint32_t)(base + j));
    __syncthreads();
    uint2* out = pairs + offsets[blockIdx.x];
    for (uint32_t j = threadIdx.x; j < total; j += 256) out[j] = buf[j];
}

// ---- exclusive scan of a uint32 array (two or three kernels) -------------------------------------------------

// The scans take an optional (info, pass): a radix pass the key range does not need is skipped by all its kernels.
__device__ __forceinline__ bool pass_skipped(const SelInfo* info, int pass) { return info && (uint32_t)pass >= info->n_passes; }
// Radix tiles that hold selected pairs (the grids and tables are sized for M == N on the host) and the length of a
// pass's digit table, 256 entries per such tile; with rtile == 0 the scan takes the length it was given.
__device__ __forceinline__ int active_tiles(const SelInfo* info, int rtile, int n_blocks) {
    const int64_t a = ((int64_t)info->M + rtile - 1) / rtile;
    return a < n_blocks ? (int)a : n_blocks;
}
__device__ __forceinline__ int64_t scan_length(int64_t n, const SelInfo* info, int rtile) {
    if (!info || rtile == 0) return n;
    const int64_t m = 256 * (((int64_t)info->M + rtile - 1) / rtile);
    return m < n ? m : n;
}

__global__ __launch_bounds__(256) void scan_chunk_sums_kernel(const uint32_t* __restrict__ data, int64_t n, uint32_t* __restrict__ sums,
                                                              const SelInfo* __restrict__ info, int pass, int rtile) {
    if (pass_skipped(info, pass)) return;
    n = scan_length(n, info, rtile);
    if ((int64_t)blockIdx.x * SCAN_CHUNK >= n) return;
    int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + threadIdx.x * 8;
    uint32_t c = 0;
    for (int j = 0; j < 8; ++j)
        if (base + j < n) c += data[base + j];
    uint32_t total;
    block_exclusive_scan_256(c, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void scan_sums_kernel(uint32_t* __restrict__ sums, int n_chunks, int64_t n, const SelInfo* __restrict__ info, int pass,
                                                        int rtile) {
    if (pass_skipped(info, pass)) return;
    n_chunks = (int)((scan_length(n, info, rtile) + SCAN_CHUNK - 1) / SCAN_CHUNK);
    uint32_t carry = 0;
    for (int b0 = 0; b0 < n_chunks; b0 += 256) {
        int i = b0 + threadIdx.x;
        uint32_t v = i < n_chunks ? sums[i] : 0u, total;
        uint32_t ex = block_exclusive_scan_256(v, &total);
        if (i < n_chunks) sums[i] = carry + ex;
        carry += total;
    }
}

// With `raw` the chunk sums have not been scanned: a workgroup adds up those before its own, a few loads per thread in place of a
// launch of one workgroup (up to SCAN_RAW_MAX chunks).
#define SCAN_RAW_MAX 4096
__global__ __launch_bounds__(256) void scan_apply_kernel(uint32_t* __restrict__ data, int64_t n, const uint32_t* __restrict__ sums,
                                                         const SelInfo* __restrict__ info, int pass, int rtile, int raw) {
    if (pass_skipped(info, pass)) return;
    n = scan_length(n, info, rtile);
    if ((int64_t)blockIdx.x * SCAN_CHUNK >= n) return;
    int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + threadIdx.x * 8;
    uint32_t v[8], c = 0;
    for (int j = 0; j < 8; ++j) {
        v[j] = base + j < n ? data[base + j] : 0u;
        c += v[j];
    }
    uint32_t before = 0;
    if (raw) {
        uint32_t mine = 0;
        for (unsigned i = threadIdx.x; i < blockIdx.x; i += 256) mine += sums[i];
        block_exclusive_scan_256(mine, &before);
    } else {
        before = sums[blockIdx.x];
    }
    uint32_t run = before + block_exclusive_scan_256(c, nullptr);
    for (int j = 0; j < 8; ++j)
        if (base + j < n) {
            data[base + j] = run;
            run += v[j];
        }
}

// The same in one launch for arrays of up to 8192 entries (block counts of pools of up to 2^24 losses; above that the
// strided per-thread loads cost more than the two launches saved): thread t of the one workgroup owns entries
// [t * per, (t + 1) * per), all loaded before anything else so that the loads overlap.
#define SCAN_ONE_LAUNCH_MAX 8192
__global__ __launch_bounds__(256) void scan_small_kernel(uint32_t* __restrict__ data, int n, int per, const SelInfo* __restrict__ info, int pass,
                                                         int rtile) {
    if (pass_skipped(info, pass)) return;
    n = (int)scan_length(n, info, rtile);
    uint32_t v[32];
    const int base = threadIdx.x * per;
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = (j < per && base + j < n) ? data[base + j] : 0u;
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) c += v[j];
    uint32_t run = block_exclusive_scan_256(c, nullptr);
#pragma unroll
    for (int j = 0; j < 32; ++j)
        if (j < per && base + j < n) {
            data[base + j] = run;
            run += v[j];
        }
}

static void exclusive_scan_u32(hipStream_t s, uint32_t* data, int64_t n, uint32_t* sums, const SelInfo* info = nullptr, int pass = 0, int rtile = 0) {
    if (n <= SCAN_ONE_LAUNCH_MAX) {
        hipLaunchKernelGGL(scan_small_kernel, dim3(1), dim3(256), 0, s, data, (int)n, (int)((n + 255) / 256), info, pass, rtile);
        return;
    }
    int n_chunks = (int)((n + SCAN_CHUNK - 1) / SCAN_CHUNK);
    hipLaunchKernelGGL(scan_chunk_sums_kernel, dim3(n_chunks), dim3(256), 0, s, data, n, sums, info, pass, rtile);
    const int raw = n_chunks <= SCAN_RAW_MAX;
    if (!raw) hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(256), 0, s, sums, n_chunks, n, info, pass, rtile);
    hipLaunchKernelGGL(scan_apply_kernel, dim3(n_chunks), dim3(256), 0, s, data, n, sums, info, pass, rtile, raw);
}

// ---- radix sort passes --------------------------------------------------------------------------------

// table[d * tiles + b] = number of elements of block b's tile with digit d, tiles = the tiles that hold pairs (active_tiles)
template <int RITER>
__global__ __launch_bounds__(256) void radix_count_kernel(const uint2* __restrict__ pairs, const SelInfo* __restrict__ info,
                                                          int shift, uint32_t* __restrict__ table, int n_blocks) {
    if ((uint32_t)(shift >> 3) >= info->n_passes) return;   // the key range does not reach these bits
    __shared__ uint32_t cnt[256];
    cnt[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t M = info->M;
    constexpr int RTILE = RITER * 256;
    int64_t base = (int64_t)blockIdx.x * RTILE;
    if (base >= M) return;   // the table only has columns for tiles that hold pairs
#pragma unroll
    for (int j = 0; j < RITER; ++j) {
        int64_t i = base + j * 256 + threadIdx.x;
        if (i < M) atomicAdd(&cnt[(pairs[i].x >> shift) & 255u], 1u);
    }
    __syncthreads();
    table[(int64_t)threadIdx.x * active_tiles(info, RTILE, n_blocks) + blockIdx.x] = cnt[threadIdx.x];
}

// table has been exclusive-scanned: table[d * n_blocks + b] = first output slot of digit d in block b.
// Each wave owns RTILE/4 consecutive elements of the tile and ranks them 64 at a time with ballots, counting every digit as it
// goes, so the order of equal digits is the input order (stable).  The pairs are then put in digit order in LDS and written out
// position by position: neighbouring lanes write neighbouring slots of a digit's run, and key and index travel as one 8-byte
// pair, so that a run of 16 fills a cache line (a pass over 4 M pairs: 25 -> 20 us).  The last pass that the key range needs
// stores the first k of the result.  With the pair layout the whole selection went from 258 to 215 us (4 M of 16 M), 608 to 473
// (all of 16 M) and 153 to 116 (all of 2^20); without a launch that unpacks the result and one per scan it takes 201, 435, 105.
template <int RITER>
__global__ __launch_bounds__(256) void radix_scatter_kernel(const uint2* __restrict__ in, uint2* __restrict__ out, const SelInfo* __restrict__ info,
                                                            int shift, const uint32_t* __restrict__ table, int n_blocks,
                                                            const float* __restrict__ losses, int64_t k, int32_t* __restrict__ idx_out,
                                                            float* __restrict__ val_out) {
    constexpr int RTILE = RITER * 256;
    __shared__ uint32_t cnt[4][256];
    __shared__ uint32_t to_global[256];   // global slot of a digit's first element minus its slot in the tile
    __shared__ uint2 buf[RTILE];
    if ((uint32_t)(shift >> 3) >= info->n_passes) return;   // the key range does not reach these bits
    const uint32_t M = info->M;
    const int64_t base = (int64_t)blockIdx.x * RTILE;
    if (base >= M) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t wbase = base + wave * (RTILE / 4);
    uint2 pair[RITER];
    uint32_t rank[RITER];
#pragma unroll
    for (int it = 0; it < RITER; ++it) {
        const int64_t i = wbase + it * 64 + lane;
        pair[it] = i < M ? in[i] : make_uint2(0u, 0u);
    }
    const uint32_t first = table[(int64_t)threadIdx.x * active_tiles(info, RTILE, n_blocks) + blockIdx.x];
#pragma unroll
    for (int w = 0; w < 4; ++w) cnt[w][threadIdx.x] = 0u;
    __syncthreads();
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
    for (int it = 0; it < RITER; ++it) {
        const bool valid = wbase + it * 64 + lane < M;
        const uint32_t d = (pair[it].x >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t v = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? v : ~v;
        }
        rank[it] = cnt[wave][d] + (uint32_t)__popcll(peers & lt);
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & lt) == 0ull) cnt[wave][d] += (uint32_t)__popcll(peers);  // lowest peer advances the count
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {   // per digit: slots of the tile in digit order, waves in order inside a digit
        uint32_t c[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) c[w] = cnt[w][threadIdx.x];
        uint32_t run = block_exclusive_scan_256((c[0] + c[1]) + (c[2] + c[3]), nullptr);
        to_global[threadIdx.x] = first - run;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            cnt[w][threadIdx.x] = run;
            run += c[w];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RITER; ++it)
        if (wbase + it * 64 + lane < M) buf[cnt[wave][(pair[it].x >> shift) & 255u] + rank[it]] = pair[it];
    __syncthreads();
    const int n_valid = (int)(M - base < (uint32_t)RTILE ? M - base : (uint32_t)RTILE);
    const bool last = (uint32_t)(shift >> 3) + 1u == info->n_passes;
    const uint32_t hi = info->hi;
    for (int j = threadIdx.x; j < n_valid; j += 256) {
        const uint2 v = buf[j];
        const uint32_t pos = to_global[(v.x >> shift) & 255u] + (uint32_t)j;
        if (!last) {
            out[pos] = v;
        } else if (pos < k) {
            idx_out[pos] = (int32_t)v.y;
            if (val_out) {
                float loss;
                if (!key_to_loss(hi - v.x, &loss)) loss = losses[v.y];
                val_out[pos] = loss;
            }
        }
    }
}

struct TopkScratch {
    uint32_t *hist, *hist2, *counts, *sums, *table;
    uint2 *a, *b;
    SelInfo* info;
    int n_blocks;    // selection tiles (TILE elements)
    int r_iter;      // rounds per wave in the radix passes (8 or 16)
    int r_blocks;    // radix tiles (r_iter * 256 elements)
};

static TopkScratch carve_topk(Carver& c, int64_t N) {
    TopkScratch t;
    t.n_blocks = (int)((N + TILE - 1) / TILE);
    t.r_iter = N >= (int64_t(1) << 22) ? 16 : 8;
    t.r_blocks = (int)((N + t.r_iter * 256 - 1) / (t.r_iter * 256));
    t.hist = c.take<uint32_t>(2 * SEL_BINS);   // both levels, cleared together
    t.hist2 = t.hist + SEL_BINS;
    t.info = c.take<SelInfo>(1);
    t.counts = c.take<uint32_t>(t.n_blocks);
    t.table = c.take<uint32_t>((size_t)256 * t.r_blocks);
    t.sums = c.take<uint32_t>(((size_t)256 * t.n_blocks + SCAN_CHUNK - 1) / SCAN_CHUNK + 1);
    t.a = c.take<uint2>(N);
    t.b = c.take<uint2>(N);
    return t;
}

size_t topk_scratch_bytes(int64_t N, int64_t k) {
    (void)k;
    if (N <= TOPK_RANK_MAX) return 0;
    Carver c(nullptr);
    if (N <= TOPK_SORT_MAX) {
        SelJob job;
        carve_sort(c, N, job);
        return c.off;
    }
    carve_topk(c, N);
    return c.off;
}

// `scratch_base`: topk_scratch_bytes(N, k) bytes of device memory, 256-byte aligned; nothing in it needs to be cleared.
static int launch_topk_large(bls_ctx* ctx, char* scratch_base, const float* losses, int64_t N, int64_t k, int32_t* idx_out, float* val_out) {
    Carver c(scratch_base);
    TopkScratch t = carve_topk(c, N);
    hipStream_t s = ctx->stream;
    const int nb = t.n_blocks, rb = t.r_blocks;
    const int64_t quads = (N + 3) / 4;
    const int64_t hist_want = (quads + HIST_THREADS - 1) / HIST_THREADS, hist_full = 2 * (int64_t)ctx->num_cus;   // 64 KB of LDS each
    const int hist_blocks = (int)(hist_want < hist_full ? hist_want : hist_full);
    const bool vec = reinterpret_cast<uintptr_t>(losses) % 16 == 0;   // 16-byte loads where the array allows them
    hipLaunchKernelGGL(zero_u32_kernel, dim3(16), dim3(256), 0, s, t.hist, (int64_t)2 * SEL_BINS);
    if (vec) hipLaunchKernelGGL((sel_hist_kernel<1, true>), dim3(hist_blocks), dim3(HIST_THREADS), 0, s, losses, N, t.info, t.hist);
    else hipLaunchKernelGGL((sel_hist_kernel<1, false>), dim3(hist_blocks), dim3(HIST_THREADS), 0, s, losses, N, t.info, t.hist);
    hipLaunchKernelGGL(sel_threshold_kernel<1>, dim3(1), dim3(256), 0, s, t.hist, (uint32_t)k, t.info);
    if (vec) hipLaunchKernelGGL((sel_hist_kernel<2, true>), dim3(hist_blocks), dim3(HIST_THREADS), 0, s, losses, N, t.info, t.hist2);
    else hipLaunchKernelGGL((sel_hist_kernel<2, false>), dim3(hist_blocks), dim3(HIST_THREADS), 0, s, losses, N, t.info, t.hist2);
    hipLaunchKernelGGL(sel_threshold_kernel<2>, dim3(1), dim3(256), 0, s, t.hist2, (uint32_t)k, t.info);
    if (vec) hipLaunchKernelGGL(sel_count_kernel<true>, dim3(nb), dim3(256), 0, s, losses, N, t.info, t.counts);
    else hipLaunchKernelGGL(sel_count_kernel<false>, dim3(nb), dim3(256), 0, s, losses, N, t.info, t.counts);
    exclusive_scan_u32(s, t.counts, nb, t.sums);
    if (vec) hipLaunchKernelGGL(sel_compact_kernel<true>, dim3(nb), dim3(256), 0, s, losses, N, t.info, t.counts, t.a);
    else hipLaunchKernelGGL(sel_compact_kernel<false>, dim3(nb), dim3(256), 0, s, losses, N, t.info, t.counts, t.a);
    uint2 *from = t.a, *to = t.b;
    for (int pass = 0; pass < 4; ++pass) {
        if (t.r_iter == 16) hipLaunchKernelGGL(radix_count_kernel<16>, dim3(rb), dim3(256), 0, s, from, t.info, pass * 8, t.table, rb);
        else hipLaunchKernelGGL(radix_count_kernel<8>, dim3(rb), dim3(256), 0, s, from, t.info, pass * 8, t.table, rb);
        exclusive_scan_u32(s, t.table, (int64_t)256 * rb, t.sums, t.info, pass, t.r_iter * 256);
        if (t.r_iter == 16) hipLaunchKernelGGL(radix_scatter_kernel<16>, dim3(rb), dim3(256), 0, s, from, to, t.info, pass * 8, t.table, rb, losses, k, idx_out, val_out);
        else hipLaunchKernelGGL(radix_scatter_kernel<8>, dim3(rb), dim3(256), 0, s, from, to, t.info, pass * 8, t.table, rb, losses, k, idx_out, val_out);
        uint2* tmp = from; from = to; to = tmp;
    }
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}

static int launch_topk_small(bls_ctx* ctx, const SelJobs& jobs, int n_jobs, int64_t N) {
    const unsigned chunks = (unsigned)((N + 63) / 64);
    const size_t words = chunks * 64 > 1024 ? chunks * 64 : 1024;   // the keys, and in their place 16 x 64 partial ranks
    hipLaunchKernelGGL(topk_rank_kernel, dim3(chunks, n_jobs), dim3(1024), words * sizeof(uint32_t), ctx->stream, jobs, (int)N);
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}

// `scratch_base`: topk_scratch_bytes(N, k) bytes of device memory, 256-byte aligned
static int launch_topk_at(bls_ctx* ctx, char* scratch_base, const float* losses, int64_t N, int64_t k, int32_t* idx_out, float* val_out) {
    if (N > TOPK_SORT_MAX) return launch_topk_large(ctx, scratch_base, losses, N, k, idx_out, val_out);
    SelJobs jobs{};
    jobs.j[0] = SelJob{losses, (int)k, idx_out, val_out, nullptr, -INFINITY};
    if (N <= TOPK_RANK_MAX) return launch_topk_small(ctx, jobs, 1, N);
    return launch_topk_medium(ctx, scratch_base, jobs, 1, N);
}

int launch_topk(bls_ctx* ctx, const float* losses, int64_t N, int64_t k, int32_t* idx_out, float* val_out) {
    int rc = bls_arena_reserve(ctx, topk_scratch_bytes(N, k));
    if (rc != BLS_OK) return rc;
    return launch_topk_at(ctx, ctx->arena, losses, N, k, idx_out, val_out);
}

// Counting beats sorting as long as its workgroups (64 samples of a selection each) run side by side; further selections share
// the chip, while those that are sorted hardly notice each other.  An epoch's draws, by counting / by sorting: one draw of 15 000
// samples 24.2 / 25.0 us, of 15 500 25.3 / 25.0; two of 8192 (a workgroup for each of 256 compute units) 15.9 / 24.3, of 9500
// 30.3 / 26.7; three of 7000 29.7 / 30.4, of 8192 33 / 30.5.
static int64_t jobs_rank_max(int n_jobs) { return n_jobs == 1 ? 15360 : n_jobs == 2 ? 8192 : 7168; }

size_t topk_jobs_scratch_bytes(int n_jobs, int64_t N) {
    if (N <= jobs_rank_max(n_jobs)) return 0;
    Carver c(nullptr);
    SelJob job;
    for (int i = 0; i < n_jobs; ++i) carve_sort(c, N, job);
    return c.off;
}

int launch_topk_jobs(bls_ctx* ctx, char* scratch_base, SelJobs jobs, int n_jobs, int64_t N) {
    return N <= jobs_rank_max(n_jobs) ? launch_topk_small(ctx, jobs, n_jobs, N) : launch_topk_medium(ctx, scratch_base, jobs, n_jobs, N);
}

// ---- selection without any allocation -----------------------------------------------------------------
//
// The large-pool path above needs device scratch (histogram, block counts, digit tables and two arrays of key and
// index).  For callers that must not allocate, the same launches run on a fixed array in the library's device image.
// Every GPU the library is loaded on holds its own copy of the array at its own address, for the life of the process.

#define TOPK_STATIC_BYTES (size_t(18) << 20)   // >= topk_scratch_bytes(BLS_TOPK_STATIC_MAX_N, .), checked on every call
#define TOPK_STATIC_MAX_DEVICES 64

static __device__ __align__(256) unsigned char scratch[TOPK_STATIC_BYTES];

// Device address of `scratch` per GPU (the array's name in host code is only a handle for the symbol lookup).
static char* g_static_scratch[TOPK_STATIC_MAX_DEVICES];
static std::mutex g_static_scratch_lock;

int topk_static_init(bls_ctx* ctx) {
    if (ctx->device < 0 || ctx->device >= TOPK_STATIC_MAX_DEVICES) return BLS_OK;   // topk_by_loss_static refuses such a device
    std::lock_guard<std::mutex> hold(g_static_scratch_lock);
    if (g_static_scratch[ctx->device]) return BLS_OK;
    void* ptr = nullptr;
    BLS_HIP(ctx, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));   // the context's device is current
    if (!ptr) return bls_fail(ctx, BLS_EHIP, "no device address for the static top-k scratch");
    g_static_scratch[ctx->device] = static_cast<char*>(ptr);
    return BLS_OK;
}

int launch_topk_static(bls_ctx* ctx, const float* losses, int64_t N, int64_t k, int32_t* idx_out, float* val_out) {
    if (N > BLS_TOPK_STATIC_MAX_N || topk_scratch_bytes(N, k) > TOPK_STATIC_BYTES)
        return bls_fail(ctx, BLS_EINVAL, "topk_by_loss_static: N = %lld exceeds the limit of %d", (long long)N, BLS_TOPK_STATIC_MAX_N);
    if (N <= TOPK_RANK_MAX) return launch_topk_at(ctx, nullptr, losses, N, k, idx_out, val_out);
    char* base = (ctx->device >= 0 && ctx->device < TOPK_STATIC_MAX_DEVICES) ? g_static_scratch[ctx->device] : nullptr;
    if (!base) return bls_fail(ctx, BLS_EUNSUPPORTED, "topk_by_loss_static: no static scratch on device %d", ctx->device);
    return launch_topk_at(ctx, base, losses, N, k, idx_out, val_out);
}
