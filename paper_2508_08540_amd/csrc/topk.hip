// Deterministic loss-based top-k selection (Section 4.2): the k highest-loss samples in rank order.
//
// Every loss is mapped to a 64-bit sort word whose unsigned order is the selection order:
//   high 32 bits: the float's bits made monotone (sign flip), with -0 folded into +0 and every
//                 NaN folded into the largest word, so NaN ranks above +inf;
//   low 32 bits:  ~index, so that among equal losses the smaller index is the larger word.
// All words are distinct, hence exactly one result is correct and no stability argument is needed.
//
// Pools of up to TOPK_RANK_MAX samples are ranked by counting in one launch; pools of up to TOPK_WHOLE_MAX are sorted whole by
// four radix passes of one launch each; larger ones take radix-select of the k-th word and an LSD radix sort of the words selected.
#include <mutex>

#include "common.h"

// Ranking by counting needs no scratch and costs 24.6 us at 16384 (four sorting passes: 22 us at 16385).  Sorting whole / selecting
// first, k = N / 50 and k = N: 200 000 samples 45 / 48 and 54 us, 262 144 (the last that four rounds of a tile hold) 51 / 48 and 55,
// 400 000 64 / 49 and 58.  (Where the keys selected range over four digits: all of 262 145 half-normal losses 57 / 61, half of 400 000 of which
// three quarters are zero 68 / 75.  Several selections in one go, TOPK_SORT_MAX, are another matter: they share the sort's launches.)
#define TOPK_RANK_MAX 16384
#define TOPK_WHOLE_MAX (1 << 18)

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

// N <= TOPK_SORT_MAX; `scratch_base` as below, n_jobs times.  The fewest rounds that keep the pool within
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
// 1. Select: a histogram of the top 14 key bits gives the bin that holds the k-th largest key.  Where that bin holds more than
//    N / 32 elements too many (they would all be sorted), a second histogram of the next 12 bits over its members gives a 26-bit
//    prefix.  The M elements with key >= thr are selected (M >= k).
// 2. Stable LSD radix sort of the M elements, 8 bits per pass, with as many passes as the range of their keys needs (the later
//    ones exit at once).  The sort key is hi - key (hi bounds every key), so that ascending order is rank order and the keys
//    only span the range that occurs.  The first pass reads the losses themselves and leaves (sort key, index) pairs; stability
//    keeps equal losses in ascending index order, which is the tie rule.
// 3. The first k pairs are the result: the last pass stores indices and losses instead of pairs.
// Nothing is read back to the host: grids are sized for the worst case M == N and blocks past M exit.
//
// A pass is two launches: digit counts of every tile, with sums over groups of SEL_GROUP tiles, and the scatter, whose
// workgroups add up the groups and the tiles of their own group before them (62 + 32 rows of 256 at 16 M keys), sixteen rows of each
// half of the threads requested at a time: in batches of eight the first pass took 56 us, now 50, and 74 with all at once, whose 156
// registers leave one workgroup per compute unit.  (Sums over 16 groups as well made its atomics meet: counts 13.6 -> 18.6 us.)
// The launches that scanned the table in between, two of 3 to 4 us and as many gaps a pass, are gone up to 2^24 samples; beyond, where adding
// up the groups would grow with the square of the pool, one launch scans their sums (SEL_GROUPS_MAX; 2 % and all of 2^25 half-normal
// losses 185 -> 163 and 928 -> 831 us, 2 % of 2^28 2.85 -> 1.01 ms, of 2^30 35.9 -> 3.9).  A compaction of
// the selected pairs before the sort (count, scan, gather: 41 us for 16 M keys) is gone too: the first pass skips what is not selected.
// 4 M of 16 M half-normal losses above ln 10: 24 launches and 201 us before, 13 and 155; all of 16 M 436 -> 330; 84 000 of 4.2 M 119 -> 74; all of
// 600 000 96 -> 59.  Pools that did better with the compaction: 2 % of 2^26 and 2^28 losses of 2.30 +- 0.03, 285 -> 325 and 1010 -> 1180 us.

#define SEL_BITS 14          // level 1
#define SEL_BINS (1 << SEL_BITS)
#define SEL_SUB 2            // counters of a bin in LDS
#define SEL_SHIFT (32 - SEL_BITS)
#define SEL_BITS2 12         // level 2
#define SEL_BINS2 (1 << SEL_BITS2)
#define SEL_SHIFT2 (SEL_SHIFT - SEL_BITS2)
#define SEL_GROUP 32         // tiles of a group of digit counts
#define SEL_GROUPS_MAX 64    // up to this many groups a scatter adds them up itself; more are scanned by a launch between
#define SEL_EXCESS 32        // level 2 runs where more than N / SEL_EXCESS elements too many would be selected

struct SelInfo {
    uint32_t thr;        // selected: key >= thr
    uint32_t M;          // number of selected elements
    uint32_t hi;         // no key is larger; sort key = hi - key
    uint32_t n_passes;   // 8-bit passes that cover hi - thr
    uint32_t above;      // elements in bins above that of thr (level 1)
    uint32_t refine;     // level 2 runs
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

// LEVEL 1: bins of the top 14 bits over all elements, 128 KB of LDS.  An octave has 32 of these bins, so that most pools do without
// level 2 (with 12 bits 4 M of 16 M half-normal losses above ln 10 need it: 157 -> 174 us).  LEVEL 2: bins of the next 12 bits over the
// members of one.
// Lanes that meet in a word are served one after the other, and losses may lie in a few bins (an untrained network's, around ln C) or be
// equal, so every bin has two counters, for odd and even lanes, and a thread adds the elements of a run in one bin at once.  2 % of
// 2^24 losses against 2^15 bins with one counter: half-normal 117 -> 116 us, 2.30 +- 0.03 151 -> 140, three quarters zero 150 -> 116, all
// within 1e-4 170 -> 124, all equal 400 -> 230.  Merging the lanes of a bin before the atomic costs every wave its ballots: the launch
// over 2^28 spread losses 250 -> 392 us.
// Workgroups of 1024 threads, one per compute unit at level 1 and two at level 2 as soon as each has eight quads a thread (2^28 losses 237 ->
// 181 us): the loop waits for memory, while every further histogram costs a clear and a fold of its bins.
#define HIST_THREADS 1024
template <int LEVEL, bool VEC>
__global__ __launch_bounds__(HIST_THREADS) void sel_hist_kernel(const float* __restrict__ losses, int64_t N, const SelInfo* __restrict__ info,
                                                       uint32_t* __restrict__ hist) {
    constexpr int BINS = LEVEL == 1 ? SEL_BINS : SEL_BINS2, SUB = LEVEL == 1 ? SEL_SUB : 1, DEPTH = 2;
    extern __shared__ __align__(16) uint32_t sel_lds[];
    if (LEVEL == 2 && !info->refine) return;
    const uint32_t b1 = LEVEL == 2 ? info->thr >> SEL_SHIFT : 0u, sub = threadIdx.x & (SUB - 1);
    for (int i = threadIdx.x; i < BINS * SUB / 4; i += HIST_THREADS) reinterpret_cast<uint4*>(sel_lds)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint32_t run_bin = 0, run = 0;   // level 1: elements of the thread since its bin last changed
    const int64_t quads = (N + 3) >> 2;
    constexpr int STRIDE = HIST_THREADS;
    for (int64_t q = (int64_t)blockIdx.x * (DEPTH * STRIDE) + threadIdx.x; q < quads; q += (int64_t)gridDim.x * (DEPTH * STRIDE)) {
        uint32_t key[DEPTH][4];
        bool ok[DEPTH][4];
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
#pragma unroll
            for (int j = 0; j < 4; ++j) ok[u][j] = false;
            if (q + u * STRIDE < quads) load_keys4<VEC>(losses, N, q + u * STRIDE, key[u], ok[u]);
        }
#pragma unroll
        for (int u = 0; u < DEPTH; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!ok[u][j]) continue;
                if (LEVEL == 1) {
                    const uint32_t bin = key[u][j] >> SEL_SHIFT;
                    if (bin != run_bin) {
                        atomicAdd(&sel_lds[run_bin * SUB + sub], run);
                        run_bin = bin;
                        run = 0;
                    }
                    ++run;
                } else if ((key[u][j] >> SEL_SHIFT) == b1) {
                    atomicAdd(&sel_lds[(key[u][j] >> SEL_SHIFT2) & (SEL_BINS2 - 1)], 1u);
                }
            }
    }
    if (LEVEL == 1) atomicAdd(&sel_lds[run_bin * SUB + sub], run);
    __syncthreads();
    for (int i = threadIdx.x; i < BINS; i += HIST_THREADS) {
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < SUB; ++u) c += sel_lds[i * SUB + u];
        if (c) atomicAdd(&hist[i], c);
    }
}

// One block: suffix counts over the bins; the bin sought is the largest one whose suffix count reaches `want`.  LEVEL 1: want = k;
// stores what follows from its bins, and whether they are too coarse.  LEVEL 2: want = k - above over the sub-bins of that bin.
template <int LEVEL>
__global__ __launch_bounds__(1024) void sel_threshold_kernel(const uint32_t* __restrict__ hist, uint32_t k, int64_t N, SelInfo* __restrict__ info) {
    constexpr int PER = (LEVEL == 1 ? SEL_BINS : SEL_BINS2) / 1024;   // bins per thread
    __shared__ uint32_t wave_total[16], top_bin;
    if (LEVEL == 2 && !info->refine) return;
    const uint32_t want = LEVEL == 1 ? k : k - info->above, first = LEVEL == 2 ? info->thr : 0u, hi_before = LEVEL == 2 ? info->hi : 0u,
                   above_before = LEVEL == 2 ? info->above : 0u;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t mine[PER], tot = 0;
    if (threadIdx.x == 0) top_bin = 0u;
#pragma unroll
    for (int j = 0; j < PER; j += 4) {
        const uint4 v = reinterpret_cast<const uint4*>(hist)[(threadIdx.x * PER + j) / 4];
        mine[j] = v.x; mine[j + 1] = v.y; mine[j + 2] = v.z; mine[j + 3] = v.w;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) tot += mine[j];
    uint32_t incl = tot;   // of this thread and the higher ones
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_down(incl, o, 64);
        if (lane + o < 64) incl += v;
    }
    if (lane == 0) wave_total[wave] = incl;
    __syncthreads();
    int top = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (mine[j]) top = j;
    if (top >= 0) atomicMax(&top_bin, (uint32_t)(threadIdx.x * PER + top));
    __syncthreads();
    uint32_t above = incl - tot;
    for (int w = wave + 1; w < 16; ++w) above += wave_total[w];
#pragma unroll
    for (int j = PER - 1; j >= 0; --j) {
        const uint32_t with = above + mine[j];
        if (above < want && with >= want) {
            const uint32_t b = threadIdx.x * PER + j;
            const uint32_t thr = LEVEL == 1 ? b << SEL_SHIFT : first | (b << SEL_SHIFT2);
            // level 1: the end of the last bin (2^32 - 1 for the largest); level 2: that of its last sub-bin where no bin is above it
            const uint32_t hi = LEVEL == 1 ? ((top_bin + 1u) << SEL_SHIFT) - 1u
                                : above_before ? hi_before : first | (((top_bin + 1u) << SEL_SHIFT2) - 1u);
            const uint32_t range = hi - thr;   // sort keys lie in [0, range]
            info->thr = thr;
            info->hi = hi;
            info->M = above_before + with;
            info->n_passes = range < 256u ? 1u : (32u - (uint32_t)__clz(range) + 7u) / 8u;   // the last pass stores the result
            if (LEVEL == 1) {
                info->above = above;
                info->refine = (int64_t)(with - want) > N / SEL_EXCESS ? 1u : 0u;
            }
        }
        above = with;
    }
}

// ---- radix sort passes --------------------------------------------------------------------------------

// Pools below 2^22: tiles of 8 rounds of 256 threads; larger ones 16 rounds of 512 (longer runs per digit when scattering,
// fewer rows to add up), whose groups may be scanned.  The smaller tiles make up at most SEL_GROUPS_MAX groups.
template <int THREADS, int RITER>
struct RadixShape {
    static constexpr int TILE = THREADS * RITER, WAVES = THREADS / 64;
    static constexpr bool SCANS = THREADS == 512;
    static __host__ __device__ int groups(int64_t elements) { return (int)((elements + (int64_t)TILE * SEL_GROUP - 1) / ((int64_t)TILE * SEL_GROUP)); }
};

// Element i of a pass as it is stored (past the end another one), the pair it sorts by, and whether it takes part.  FIRST: losses.
template <bool FIRST>
__device__ __forceinline__ uint2 radix_load(const uint2* __restrict__ pairs, const float* __restrict__ losses, int64_t N, uint32_t M, int64_t i) {
    if (FIRST) return make_uint2(__float_as_uint(losses[i < N ? i : N - 1]), 0u);
    return pairs[i < (int64_t)M ? i : 0];
}
template <bool FIRST>
__device__ __forceinline__ bool radix_take(uint2& pair, int64_t N, uint32_t M, uint32_t thr, uint32_t hi, int64_t i) {
    if (!FIRST) return i < (int64_t)M;
    const uint32_t key = loss_key(__uint_as_float(pair.x));
    pair = make_uint2(hi - key, (uint32_t)i);
    return i < N && key >= thr;
}

// table[tile][d] = number of elements of the tile with digit d, group[tile / SEL_GROUP][d] = their sums (cleared beforehand)
template <int THREADS, int RITER, bool FIRST>
__global__ __launch_bounds__(THREADS) void radix_count_kernel(const uint2* __restrict__ pairs, const float* __restrict__ losses, int64_t N,
                                                              const SelInfo* __restrict__ info, int shift, uint32_t* __restrict__ table,
                                                              uint32_t* __restrict__ group) {
    if ((uint32_t)(shift >> 3) >= info->n_passes) return;   // the key range does not reach these bits
    __shared__ uint32_t cnt[256];
    const uint32_t M = info->M, thr = info->thr, hi = info->hi;
    const int64_t base = (int64_t)blockIdx.x * RadixShape<THREADS, RITER>::TILE;
    if (!FIRST && base >= M) return;
    uint2 pair[RITER];
    bool ok[RITER];
#pragma unroll
    for (int j = 0; j < RITER; ++j) pair[j] = radix_load<FIRST>(pairs, losses, N, M, base + j * THREADS + threadIdx.x);
    if (threadIdx.x < 256) cnt[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RITER; ++j) ok[j] = radix_take<FIRST>(pair[j], N, M, thr, hi, base + j * THREADS + threadIdx.x);
#pragma unroll
    for (int j = 0; j < RITER; ++j)
        if (ok[j]) atomicAdd(&cnt[(pair[j].x >> shift) & 255u], 1u);
    __syncthreads();
    if (threadIdx.x < 256) {
        const uint32_t c = cnt[threadIdx.x];
        table[(int64_t)blockIdx.x * 256 + threadIdx.x] = c;
        if (c) atomicAdd(&group[(int64_t)(blockIdx.x / SEL_GROUP) * 256 + threadIdx.x], c);
    }
}

// More than SEL_GROUPS_MAX groups: every row of sums becomes that of the groups before it, and row `total_row` that of all of them
// (a scatter that adds up the rows itself reads as much as the square of the pool).  A workgroup takes 16 digits, a thread a 64th
// of the groups of one.
template <class Shape, bool FIRST>
__global__ __launch_bounds__(1024) void radix_scan_kernel(const SelInfo* __restrict__ info, int64_t N, int shift, uint32_t* __restrict__ group, int total_row) {
    __shared__ uint32_t part[64][16];
    if ((uint32_t)(shift >> 3) >= info->n_passes) return;
    const int groups = Shape::groups(FIRST ? N : (int64_t)info->M);
    if (groups <= SEL_GROUPS_MAX) return;
    const int c = threadIdx.x & 15, sl = threadIdx.x >> 4, per = (groups + 63) >> 6;
    const int g0 = min(sl * per, groups), g1 = min(g0 + per, groups);
    uint32_t* col = group + blockIdx.x * 16 + c;
    uint32_t sum = 0;
#pragma unroll 8
    for (int g = g0; g < g1; ++g) sum += col[(int64_t)g * 256];
    part[sl][c] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int s = 0; s < sl; ++s) run += part[s][c];
    if (sl == 63) col[(int64_t)total_row * 256] = run + sum;
    for (int g = g0; g < g1; g += 8) {
        uint32_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = g + j < g1 ? col[(int64_t)(g + j) * 256] : 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (g + j < g1) {
                col[(int64_t)(g + j) * 256] = run;
                run += v[j];
            }
    }
}

// Each wave owns RITER * 64 consecutive elements of the tile and ranks them 64 at a time with ballots, counting every digit as it
// goes, so the order of equal digits is the input order (stable).  The pairs are then put in digit order in LDS and written out
// position by position: neighbouring lanes write neighbouring slots of a digit's run, and key and index travel as one 8-byte
// pair, so that a run of 16 fills a cache line (a pass over 4 M pairs: 25 -> 20 us).  The last pass that the key range needs
// stores the first k of the result.
template <int THREADS, int RITER, bool FIRST>
__global__ __launch_bounds__(THREADS, 4) void radix_scatter_kernel(const uint2* __restrict__ in, uint2* __restrict__ out, int64_t N,
                                                                const SelInfo* __restrict__ info, int shift, const uint32_t* __restrict__ table,
                                                                const uint32_t* __restrict__ group, int total_row, const float* __restrict__ losses, int64_t k,
                                                                int32_t* __restrict__ idx_out, float* __restrict__ val_out) {
    constexpr int TILE = RadixShape<THREADS, RITER>::TILE, WAVES = RadixShape<THREADS, RITER>::WAVES;
    __shared__ uint32_t cnt[WAVES][256];
    __shared__ uint32_t to_global[256];   // global slot of a digit's first element minus its slot in the tile
    __shared__ uint32_t part[2][WAVES / 4][256];
    __shared__ uint32_t wave_total[2][4];
    __shared__ uint2 buf[TILE];
    if ((uint32_t)(shift >> 3) >= info->n_passes) return;   // the key range does not reach these bits
    const uint32_t M = info->M, thr = info->thr, hi = info->hi;
    const bool last = (uint32_t)(shift >> 3) + 1u == info->n_passes;
    const int64_t base = (int64_t)blockIdx.x * TILE;
    if (!FIRST && base >= M) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t wbase = base + wave * (RITER * 64);
    uint2 pair[RITER];
    uint32_t rank[RITER];
    bool ok[RITER];
#pragma unroll
    for (int it = 0; it < RITER; ++it) pair[it] = radix_load<FIRST>(in, losses, N, M, wbase + it * 64 + lane);
    {   // a digit's elements in all tiles, and in those before this one
        constexpr int SLICES = WAVES / 4;
        const int d = threadIdx.x & 255, g0 = threadIdx.x >> 8, tile = blockIdx.x;
        const int groups = RadixShape<THREADS, RITER>::groups(FIRST ? N : (int64_t)M), own = tile / SEL_GROUP;
        uint32_t v[SEL_GROUP / SLICES], all = 0, left = 0;
#pragma unroll
        for (int j = 0; j < SEL_GROUP / SLICES; ++j) {
            const int t = own * SEL_GROUP + g0 + SLICES * j;
            v[j] = t < tile ? table[(int64_t)t * 256 + d] : 0u;
        }
        const bool scanned = RadixShape<THREADS, RITER>::SCANS && groups > SEL_GROUPS_MAX;
        if (scanned && g0 == 0) {
            all = group[(int64_t)total_row * 256 + d];
            left = group[(int64_t)own * 256 + d];
        }
        for (int q = scanned ? groups : g0; q < groups; q += 16 * SLICES) {
            uint32_t w[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) w[j] = q + SLICES * j < groups ? group[(int64_t)(q + SLICES * j) * 256 + d] : 0u;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                all += w[j];
                left += q + SLICES * j < own ? w[j] : 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < SEL_GROUP / SLICES; ++j) left += v[j];
        part[0][g0][d] = all;
        part[1][g0][d] = left;
    }
    for (int i = threadIdx.x; i < WAVES * 256; i += THREADS) cnt[i >> 8][i & 255] = 0u;
#pragma unroll
    for (int it = 0; it < RITER; ++it) ok[it] = radix_take<FIRST>(pair[it], N, M, thr, hi, wbase + it * 64 + lane);   // waits for the loads
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    int rounds = RITER;
    if constexpr (FIRST) {
        // the selected elements of the wave side by side, in order: rounds that rank nothing are skipped
        uint2* own = buf + wave * (RITER * 64);
        int n = 0;
#pragma unroll
        for (int it = 0; it < RITER; ++it) {
            const uint64_t sel = __ballot(ok[it]);
            if (ok[it]) own[n + __popcll(sel & lt)] = pair[it];
            n += __popcll(sel);
        }
        __builtin_amdgcn_wave_barrier();
        rounds = (n + 63) >> 6;
#pragma unroll
        for (int it = 0; it < RITER; ++it) {
            ok[it] = it * 64 + lane < n;
            pair[it] = own[it * 64 + lane];   // past the n-th: not used
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RITER; ++it) {
        rank[it] = 0;
        if (!FIRST || it < rounds) {
            const bool valid = ok[it];
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
    }
    __syncthreads();
    // thread d < 256: slots of the tile in digit order, waves in order inside a digit, and the digit's first global slot
    uint32_t c[WAVES], mine = 0, total = 0, in_mine = 0, in_total = 0;
    if (threadIdx.x < 256) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            c[w] = cnt[w][threadIdx.x];
            mine += c[w];
        }
#pragma unroll
        for (int g = 0; g < WAVES / 4; ++g) total += part[0][g][threadIdx.x];
        in_mine = mine;
        in_total = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t a = __shfl_up(in_mine, o, 64), b = __shfl_up(in_total, o, 64);
            if (lane >= o) {
                in_mine += a;
                in_total += b;
            }
        }
        if (lane == 63) {
            wave_total[0][wave] = in_mine;
            wave_total[1][wave] = in_total;
        }
    }
    __syncthreads();
    int n_valid = (int)((wave_total[0][0] + wave_total[0][1]) + (wave_total[0][2] + wave_total[0][3]));
    if (threadIdx.x < 256) {
        uint32_t run = in_mine - mine, first = in_total - total;
        for (int w = 0; w < wave; ++w) {
            run += wave_total[0][w];
            first += wave_total[1][w];
        }
#pragma unroll
        for (int g = 0; g < WAVES / 4; ++g) first += part[1][g][threadIdx.x];
        to_global[threadIdx.x] = first - run;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            cnt[w][threadIdx.x] = run;
            run += c[w];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RITER; ++it)
        if (ok[it]) buf[cnt[wave][(pair[it].x >> shift) & 255u] + rank[it]] = pair[it];
    __syncthreads();
    for (int j = threadIdx.x; j < n_valid; j += THREADS) {
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
    uint32_t *hist, *hist2, *sums, *table;   // the first three are cleared together; sums: of groups, and of all of them, per pass
    uint2 *a, *b;
    SelInfo* info;
    int64_t cleared;
    bool big;        // tiles of 16 x 512 elements instead of 8 x 256
    int tiles, groups;
};

static TopkScratch carve_topk(Carver& c, int64_t N) {
    TopkScratch t;
    t.big = N >= (int64_t(1) << 22);
    t.tiles = (int)ceil_div(N, t.big ? RadixShape<512, 16>::TILE : RadixShape<256, 8>::TILE);
    t.groups = (int)ceil_div(t.tiles, SEL_GROUP);   // at most SEL_GROUPS_MAX unless big
    t.cleared = SEL_BINS + SEL_BINS2 + (int64_t)4 * (t.groups + 1) * 256;
    t.hist = c.take<uint32_t>(t.cleared);
    t.hist2 = t.hist + SEL_BINS;
    t.sums = t.hist2 + SEL_BINS2;
    t.info = c.take<SelInfo>(1);
    t.table = c.take<uint32_t>((size_t)256 * t.tiles);
    t.a = c.take<uint2>(N);
    t.b = c.take<uint2>(N);
    return t;
}

template <int THREADS, int RITER>
static void launch_radix(hipStream_t s, const TopkScratch& t, const float* losses, int64_t N, int64_t k, int32_t* idx_out, float* val_out) {
    using Shape = RadixShape<THREADS, RITER>;
    const dim3 grid(t.tiles), threads(THREADS);
    uint2 *from = t.b, *to = t.a;
    for (int pass = 0; pass < 4; ++pass) {
        uint32_t* group = t.sums + (int64_t)pass * (t.groups + 1) * 256;
#define RADIX_PASS(FIRST)                                                                                                                       \
    do {                                                                                                                                        \
        hipLaunchKernelGGL((radix_count_kernel<THREADS, RITER, FIRST>), grid, threads, 0, s, from, losses, N, t.info, pass * 8, t.table, group); \
        if constexpr (Shape::SCANS)                                                                                                             \
            if (t.groups > SEL_GROUPS_MAX)                                                                                                      \
                hipLaunchKernelGGL((radix_scan_kernel<Shape, FIRST>), dim3(16), dim3(1024), 0, s, t.info, N, pass * 8, group, t.groups);        \
        hipLaunchKernelGGL((radix_scatter_kernel<THREADS, RITER, FIRST>), grid, threads, 0, s, from, to, N, t.info, pass * 8, t.table, group,   \
                           t.groups, losses, k, idx_out, val_out);                                                                              \
    } while (0)
        if (pass == 0) RADIX_PASS(true);
        else RADIX_PASS(false);
#undef RADIX_PASS
        uint2* tmp = from; from = to; to = tmp;
    }
}

size_t topk_scratch_bytes(int64_t N, int64_t k) {
    (void)k;
    if (N <= TOPK_RANK_MAX) return 0;
    Carver c(nullptr);
    if (N <= TOPK_WHOLE_MAX) {
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
    const int64_t hist_most = ceil_div(ceil_div(N, 4), HIST_THREADS);
    auto hist_blocks = [&](int level) {
        int64_t n = ctx->num_cus;
        if (level == 2 && hist_most > 8 * n) n = hist_most < 16 * n ? hist_most / 8 : 2 * n;
        return (unsigned)(hist_most < n ? hist_most : n);
    };
    const bool vec = reinterpret_cast<uintptr_t>(losses) % 16 == 0;   // 16-byte loads where the array allows them
    hipLaunchKernelGGL(zero_u32_kernel, dim3(256), dim3(256), 0, s, t.hist, t.cleared);
#define SEL_HIST(LEVEL, VEC, HIST) \
    hipLaunchKernelGGL((sel_hist_kernel<LEVEL, VEC>), dim3(hist_blocks(LEVEL)), dim3(HIST_THREADS), 4 * (LEVEL == 1 ? SEL_BINS * SEL_SUB : SEL_BINS2), s, losses, N, t.info, HIST)
    if (vec) SEL_HIST(1, true, t.hist);
    else SEL_HIST(1, false, t.hist);
    hipLaunchKernelGGL(sel_threshold_kernel<1>, dim3(1), dim3(1024), 0, s, t.hist, (uint32_t)k, N, t.info);
    if (vec) SEL_HIST(2, true, t.hist2);
    else SEL_HIST(2, false, t.hist2);
#undef SEL_HIST
    hipLaunchKernelGGL(sel_threshold_kernel<2>, dim3(1), dim3(1024), 0, s, t.hist2, (uint32_t)k, N, t.info);
    if (t.big) launch_radix<512, 16>(s, t, losses, N, k, idx_out, val_out);
    else launch_radix<256, 8>(s, t, losses, N, k, idx_out, val_out);
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
    if (N > TOPK_WHOLE_MAX) return launch_topk_large(ctx, scratch_base, losses, N, k, idx_out, val_out);
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
// The paths above need device scratch (histograms, digit tables and their sums, two arrays of key and index).  For callers that
// must not allocate, the same launches run on a fixed array in the library's device image.
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
