// Epoch sampler (Section 4.2; the sampling steps that open every epoch of Algorithm 1), composed on the
// device from the top-k selection: the high-loss part is a top-k of the losses, uniform sampling without
// replacement of m items is the top-m of one random key per sample, and "the rest of the data" is the order of all
// keys without the samples that are already taken.  That order does not depend on what is taken, so pools of up to
// TOPK_SORT_MAX samples are ranked for the three draws in the same launches, and two more launches walk the orders that have to
// leave samples out.  Larger pools fill the chip with one selection: there the draws follow one another, and the keys
// of samples already taken are overwritten with -inf before the next one.
#include "common.h"

// Copy of the caller's keys that the exclusion below writes into.  Keys are finite by contract; a key of -inf is lifted
// to the lowest finite value so that it still ranks above the struck entries and a struck sample is never drawn again.
__global__ __launch_bounds__(256) void copy_keys_kernel(const float* __restrict__ src, float* __restrict__ dst, int64_t n) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float v = src[i];
        dst[i] = v == -INFINITY ? -3.402823466e38f : v;
    }
}

__global__ __launch_bounds__(256) void exclude_selected_kernel(const int32_t* __restrict__ sel, int64_t k, float* __restrict__ keys) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < k; i += stride) keys[sel[i]] = -INFINITY;
}

// Round-robin dealing: rank r goes to worker r % P, position r / P of that worker's contiguous segment.
// The first n % P workers hold one element more.
struct DealGroup {
    const int32_t* ranked;
    int64_t n;
    int P;
    int32_t* out;
};
__global__ __launch_bounds__(256) void deal_kernel(DealGroup first, DealGroup second) {   // blockIdx.y: the group
    const DealGroup& grp = blockIdx.y ? second : first;
    const int64_t n = grp.n;
    const int P = grp.P;
    const int32_t* __restrict__ ranked = grp.ranked;
    int32_t* __restrict__ out = grp.out;
    const int64_t base = n / P, rem = n % P;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
        const int64_t p = r % P, j = r / P;
        out[p * base + (p < rem ? p : rem) + j] = ranked[r];
    }
}

__device__ __forceinline__ uint32_t deal_slot(uint32_t n, uint32_t P, uint32_t r) {
    const uint32_t base = n / P, rem = n - base * P, j = r / P, p = r - j * P;
    return p * base + (p < rem ? p : rem) + j;
}

// Order of all samples by their key, of which the first `want` that are not chosen yet are drawn, in that order: rank `first` on
// of the group `out` is dealt to.
struct DrawJob {
    const int32_t* order;
    uint8_t* chosen;
    uint32_t* counts;        // per tile of DRAW_TILE places: samples that are not chosen
    const int32_t* ranked;   // ranks 0 .. first - 1 of the group, dealt here as well
    int32_t* out;
    uint32_t N, n, P, first, want;
    int mark;                // the drawn samples become chosen ones
};
#define DRAW_PER_THREAD 4
#define DRAW_TILE (256 * DRAW_PER_THREAD)

__device__ __forceinline__ uint32_t draw_scan_256(uint32_t v, uint32_t* wave_total, uint32_t* total) {   // exclusive
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
    *total = (wave_total[0] + wave_total[1]) + (wave_total[2] + wave_total[3]);
    return before + incl - v;
}

__device__ __forceinline__ uint32_t draw_load(const DrawJob& job, uint32_t (&id)[DRAW_PER_THREAD], bool (&free)[DRAW_PER_THREAD]) {
    const uint32_t at = blockIdx.x * DRAW_TILE + threadIdx.x * DRAW_PER_THREAD;
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < DRAW_PER_THREAD; ++j) id[j] = at + j < job.N ? (uint32_t)job.order[at + j] : 0u;
#pragma unroll
    for (int j = 0; j < DRAW_PER_THREAD; ++j) {
        free[j] = at + j < job.N && !job.chosen[id[j]];
        c += free[j];
    }
    return c;
}

__global__ __launch_bounds__(256) void draw_count_kernel(DrawJob job) {
    __shared__ uint32_t wave_total[4];
    uint32_t id[DRAW_PER_THREAD], total;
    bool free[DRAW_PER_THREAD];
    draw_scan_256(draw_load(job, id, free), wave_total, &total);
    if (threadIdx.x == 0) job.counts[blockIdx.x] = total;
}

// blockIdx.y == 1 deals the other group, whose ranks are there already
__global__ __launch_bounds__(256) void draw_kernel(DrawJob job, DealGroup other) {
    const uint32_t thread = blockIdx.x * 256 + threadIdx.x, threads = gridDim.x * 256;
    if (blockIdx.y) {
        for (uint32_t r = thread; r < (uint32_t)other.n; r += threads) other.out[deal_slot((uint32_t)other.n, other.P, r)] = other.ranked[r];
        return;
    }
    __shared__ uint32_t wave_total[2][4];
    for (uint32_t r = thread; r < job.first; r += threads) job.out[deal_slot(job.n, job.P, r)] = job.ranked[r];
    uint32_t before = 0, total;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += 256) before += job.counts[t];
    uint32_t id[DRAW_PER_THREAD];
    bool free[DRAW_PER_THREAD];
    const uint32_t c = draw_load(job, id, free);
    draw_scan_256(before, wave_total[0], &total);
    uint32_t dummy, r = total + draw_scan_256(c, wave_total[1], &dummy);
#pragma unroll
    for (int j = 0; j < DRAW_PER_THREAD; ++j) {
        if (!free[j]) continue;
        if (r < job.want) {
            job.out[deal_slot(job.n, job.P, job.first + r)] = (int32_t)id[j];
            if (job.mark) job.chosen[id[j]] = 1;   // every sample has one place in the order: no other thread asks for it in this launch
        }
        ++r;
    }
}

static unsigned blocks_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

// Pools of up to TOPK_SORT_MAX samples; see launch_sample_epoch.  50 000 samples, three draws: 66 -> 47 us, twelve launches -> seven (16 384:
// 78 -> 32, 2^19: 173 -> 132).
static int sample_epoch_together(bls_ctx* ctx, const float* losses, const float* u_biased, const float* u_other, int64_t N, int64_t n_biased,
                                 int64_t k, int64_t n_other, int P_biased, int P_other, bool unified, int32_t* biased_out, int32_t* other_out) {
    if (k > n_biased) k = n_biased;
    const bool rest = n_biased > k, after_loss = k > 0 && rest;   // keys draw the rest of the first group, without the by-loss part
    const bool other_after = unified && n_biased > 0 && n_other > 0;
    auto take = [&](Carver& c, size_t bytes) { return c.take<char>(bytes); };
    Carver sizes(nullptr);
    const size_t tiles = (size_t)ceil_div(N, DRAW_TILE);
    char* part[6];
    auto carve = [&](Carver& c) {
        part[0] = take(c, topk_jobs_scratch_bytes(3, N));
        for (int i = 1; i < 4; ++i) part[i] = take(c, sizeof(int32_t) * (size_t)N);
        part[4] = take(c, (size_t)N);
        part[5] = take(c, sizeof(uint32_t) * tiles);
    };
    carve(sizes);
    int rc = bls_arena_reserve(ctx, sizes.off);
    if (rc != BLS_OK) return rc;
    Carver c(ctx->arena);
    carve(c);
    int32_t *ranked = reinterpret_cast<int32_t*>(part[1]), *order = reinterpret_cast<int32_t*>(part[2]), *ranked_other = reinterpret_cast<int32_t*>(part[3]);
    uint8_t* chosen = reinterpret_cast<uint8_t*>(part[4]);
    uint32_t* counts = reinterpret_cast<uint32_t*>(part[5]);
    // keys are finite by contract; where others are left out, one of -inf ranks with the lowest float
    constexpr float NONE = -INFINITY, LOWEST = -3.402823466e38f;
    SelJobs jobs{};
    int n = 0;
    if (k > 0) jobs.j[n++] = SelJob{losses, (int)k, ranked, nullptr, after_loss || other_after ? chosen : nullptr, NONE};
    if (after_loss) jobs.j[n++] = SelJob{u_biased, (int)N, order, nullptr, nullptr, LOWEST};
    else if (rest) jobs.j[n++] = SelJob{u_biased, (int)n_biased, ranked, nullptr, other_after ? chosen : nullptr, NONE};
    if (n_other > 0) jobs.j[n++] = other_after ? SelJob{u_other, (int)N, ranked_other, nullptr, nullptr, LOWEST} : SelJob{u_other, (int)n_other, ranked_other, nullptr, nullptr, NONE};
    if (n == 0) return BLS_OK;
    rc = launch_topk_jobs(ctx, part[0], jobs, n, N);
    if (rc != BLS_OK) return rc;
    hipStream_t s = ctx->stream;
    const DealGroup first{ranked, n_biased, P_biased, biased_out}, second{ranked_other, n_other, P_other, other_out};
    auto draw = [&](const DrawJob& job, const DealGroup* beside) {
        hipLaunchKernelGGL(draw_count_kernel, dim3((unsigned)tiles), dim3(256), 0, s, job);
        hipLaunchKernelGGL(draw_kernel, dim3((unsigned)tiles, beside ? 2 : 1), dim3(256), 0, s, job, beside ? *beside : DealGroup{});
    };
    const bool other_ready = n_other > 0 && !other_after;
    if (after_loss)
        draw(DrawJob{order, chosen, counts, ranked, biased_out, (uint32_t)N, (uint32_t)n_biased, (uint32_t)P_biased, (uint32_t)k, (uint32_t)(n_biased - k), other_after},
             other_ready ? &second : nullptr);
    if (other_after)
        draw(DrawJob{ranked_other, chosen, counts, nullptr, other_out, (uint32_t)N, (uint32_t)n_other, (uint32_t)P_other, 0u, (uint32_t)n_other, 0},
             n_biased > 0 && !after_loss ? &first : nullptr);
    if (!after_loss && !other_after) {
        if (n_biased > 0 && n_other > 0)
            hipLaunchKernelGGL(deal_kernel, dim3(blocks_for(n_biased > n_other ? n_biased : n_other), 2), dim3(256), 0, s, first, second);
        else if (n_biased > 0) hipLaunchKernelGGL(deal_kernel, dim3(blocks_for(n_biased)), dim3(256), 0, s, first, first);
        else hipLaunchKernelGGL(deal_kernel, dim3(blocks_for(n_other)), dim3(256), 0, s, second, second);
    }
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}

// The by-loss group takes the k highest losses, then n_biased - k by its own key from the rest; the other group takes
// n_other by its key from all N (separated) or from what the first group left (unified: the first group's picks are
// struck from the other group's keys as well).
int launch_sample_epoch(bls_ctx* ctx, const float* losses, const float* u_biased, const float* u_other, int64_t N, int64_t n_biased,
                        int64_t k, int64_t n_other, int P_biased, int P_other, bool unified, int32_t* biased_out, int32_t* other_out) {
    if (N <= TOPK_SORT_MAX)
        return sample_epoch_together(ctx, losses, u_biased, u_other, N, n_biased, k, n_other, P_biased, P_other, unified, biased_out, other_out);
    // scratch: the selection's own region first (it carves from the arena base), then the masked keys and the ranking
    const size_t topk_bytes = (topk_scratch_bytes(N, N) + 255) & ~size_t(255);
    Carver sizes(nullptr);
    sizes.take<float>(N);
    sizes.take<int32_t>(N);
    sizes.take<int32_t>(N);
    int rc = bls_arena_reserve(ctx, topk_bytes + sizes.off);
    if (rc != BLS_OK) return rc;
    Carver c(ctx->arena + topk_bytes);
    float* keys = c.take<float>(N);
    int32_t* ranked = c.take<int32_t>(N);
    int32_t* ranked_other = c.take<int32_t>(N);
    hipStream_t s = ctx->stream;
    if (n_biased > 0) {
        if (k > 0) {
            rc = launch_topk(ctx, losses, N, k, ranked, nullptr);
            if (rc != BLS_OK) return rc;
        }
        if (n_biased > k) {
            const float* from = u_biased;   // nothing to strike when no sample was taken by loss
            if (k > 0) {
                hipLaunchKernelGGL(copy_keys_kernel, dim3(blocks_for(N)), dim3(256), 0, s, u_biased, keys, N);
                hipLaunchKernelGGL(exclude_selected_kernel, dim3(blocks_for(k)), dim3(256), 0, s, ranked, k, keys);
                from = keys;
            }
            rc = launch_topk(ctx, from, N, n_biased - k, ranked + k, nullptr);
            if (rc != BLS_OK) return rc;
        }
    }
    if (n_other > 0) {
        const float* from = u_other;
        if (unified && n_biased > 0) {
            hipLaunchKernelGGL(copy_keys_kernel, dim3(blocks_for(N)), dim3(256), 0, s, u_other, keys, N);
            hipLaunchKernelGGL(exclude_selected_kernel, dim3(blocks_for(n_biased)), dim3(256), 0, s, ranked, n_biased, keys);
            from = keys;
        }
        rc = launch_topk(ctx, from, N, n_other, ranked_other, nullptr);
        if (rc != BLS_OK) return rc;
    }
    const DealGroup groups[2] = {{ranked, n_biased, P_biased, biased_out}, {ranked_other, n_other, P_other, other_out}};
    if (n_biased > 0 && n_other > 0)
        hipLaunchKernelGGL(deal_kernel, dim3(blocks_for(n_biased > n_other ? n_biased : n_other), 2), dim3(256), 0, s, groups[0], groups[1]);
    else if (n_biased > 0) hipLaunchKernelGGL(deal_kernel, dim3(blocks_for(n_biased)), dim3(256), 0, s, groups[0], groups[0]);
    else if (n_other > 0) hipLaunchKernelGGL(deal_kernel, dim3(blocks_for(n_other)), dim3(256), 0, s, groups[1], groups[1]);
    BLS_HIP(ctx, hipGetLastError());
    return BLS_OK;
}
