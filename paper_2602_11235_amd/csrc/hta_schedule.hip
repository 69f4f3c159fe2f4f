// Work schedule of a jagged batch, built on the device from hist_len / n_targets (no host round trip).
//
// Under the hybrid mask (rules 1 and 3, Section 3.2.2) user b owns exactly the tiles
// (query rows) x (history keys): rows = L_b + T_b in a full layer, T_b in a target layer, keys = L_b
// (with real-time tokens, rule 2, their keys and rows count like history ones);
// nothing else is ever issued (the self key of a target row is a per-row term).  The attention
// kernels enumerate those tiles from (L_b, T_b) themselves; what the schedule adds is the ORDER of
// the users: workgroups are dispatched user-major, so listing users by decreasing tile count
// (rows x keys) starts the long-history users first and leaves the short ones to fill the tail.
#include "hta_common.h"
#include "hta_rows.h"

#include <algorithm>

namespace hta {
namespace {

constexpr int SCHED_THREADS = 1024;  // of the bucketed sort
constexpr int RANK_SORT_MAX = 4096;   // exact, deterministic rank sort up to this many users
constexpr int N_BUCKETS = 2048;       // bucketed counting sort above it

// tiles a user owns: (query rows) x (keys that run through the tile loops: history, then real-time tokens)
__device__ inline float user_cost(const Params& p, int b) {
    const float L = (float)p.hist_len[b] + (p.rt_len ? (float)p.rt_len[b] : 0.f), T = (float)p.n_targets[b];
    return (p.layer == 0 ? L + T : T) * L;
}

// order[i] = user with the i-th largest cost; ties broken by user index, so the result is unique.  The kernel is all latency, and
// runs twice in a training step: a workgroup ranks RANK_USERS users against all, RANK_LANES lanes to a user, instead of one
// workgroup with a lane to a user that walks the whole batch (64 users 4.9 -> 3.9 us, 256 users 9.0 -> 4.7, 512 users 4.7 and 4096 15.0 now).
constexpr int RANK_THREADS = 256, RANK_LANES = 16, RANK_USERS = RANK_THREADS / RANK_LANES;
static_assert(QUEUE_WORDS <= RANK_THREADS, "the first workgroup clears the counters");
// The workgroups behind the first n_rank find the rows' limits of mask rule 2, limit_groups to a user: with real-time tokens a call needs
// both before its first attention kernel, and neither needs the other (whole steps
// against a launch for each: 32 users of 60..250 keys 61.7 -> 57.7 us, 200 target layers of 250..1000 keys 153.6 -> 148.9).
__global__ __launch_bounds__(RANK_THREADS) void schedule_rank_kernel(Params p, int32_t* counters, int32_t* order, unsigned n_rank,
                                                                     unsigned limit_groups) {
    __shared__ float cost[RANK_SORT_MAX];
    const int B = p.batch, tid = threadIdx.x;
    if (blockIdx.x >= n_rank) {
        const unsigned id = blockIdx.x - n_rank, b = id / limit_groups;
        rt_limit_of_row(p, (int)b, (int)(id - b * limit_groups) * RANK_THREADS + tid);
        return;
    }
    if (blockIdx.x == 0 && tid < QUEUE_WORDS) counters[tid] = 0;
    for (int b = tid; b < B; b += RANK_THREADS) cost[b] = user_cost(p, b);
    __syncthreads();
    const int b = blockIdx.x * RANK_USERS + tid / RANK_LANES, l = tid % RANK_LANES;
    const float c = cost[min(b, B - 1)];
    int rank = 0;
#pragma unroll 4
    for (int o = l; o < B; o += RANK_LANES) {
        const float co = cost[o];
        rank += (co > c || (co == c && o < b)) ? 1 : 0;
    }
#pragma unroll
    for (int m = RANK_LANES / 2; m > 0; m /= 2) rank += __shfl_xor(rank, m);
    if (l == 0 && b < B) order[rank] = b;
}

// Large batches: users fall into N_BUCKETS cost classes (by cost / max possible cost); classes are laid out
// by decreasing cost, users inside a class in arrival order of the atomics (any order is a valid schedule).
__global__ __launch_bounds__(SCHED_THREADS) void schedule_bucket_kernel(Params p, int32_t* counters, int32_t* order) {
    __shared__ int count[N_BUCKETS];
    __shared__ int start[N_BUCKETS];
    const int B = p.batch;
    if (threadIdx.x < QUEUE_WORDS) counters[threadIdx.x] = 0;
    const float keys_max = (float)max_lead_keys(p);
    const float rows_max = p.layer == 0 ? keys_max + (float)p.max_targets : (float)p.max_targets;
    const float inv = (float)(N_BUCKETS - 1) / fmaxf(rows_max * keys_max, 1.f);
    for (int i = threadIdx.x; i < N_BUCKETS; i += SCHED_THREADS) count[i] = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += SCHED_THREADS) {
        const int k = min(N_BUCKETS - 1, max(0, (int)(user_cost(p, b) * inv)));
        atomicAdd(&count[N_BUCKETS - 1 - k], 1);  // bucket 0 = most expensive class
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int i = 0; i < N_BUCKETS; i++) {
            start[i] = acc;
            acc += count[i];
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += SCHED_THREADS) {
        const int k = min(N_BUCKETS - 1, max(0, (int)(user_cost(p, b) * inv)));
        order[atomicAdd(&start[N_BUCKETS - 1 - k], 1)] = b;
    }
}

__global__ __launch_bounds__(256) void rt_limits_kernel(Params p) { rt_limit_of_row(p, blockIdx.z, blockIdx.x * 256 + threadIdx.x); }

// bf16 heads of 16 features ride the 32-wide matrix tiles zero-padded: rows [n][16] <-> [n][32] with the upper half
// zero (one thread per 16-byte chunk).  Zero features change no score and no gradient of the features that exist.
__global__ __launch_bounds__(256) void widen16_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n_rows) {
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;  // chunk of the wide row
    if (id >= n_rows * 4) return;
    const int64_t row = id >> 2;
    const int c = (int)(id & 3);
    dst[id] = c < 2 ? src[row * 2 + c] : uint4{0u, 0u, 0u, 0u};
}
__global__ __launch_bounds__(256) void narrow16_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n_rows) {
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;  // chunk of the narrow row
    if (id >= n_rows * 2) return;
    dst[id] = src[(id >> 1) * 4 + (id & 1)];
}

}  // namespace

hipError_t launch_widen16(const void* src, void* dst, int64_t n_rows, hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(widen16_kernel, dim3((unsigned)((n_rows * 4 + 255) / 256)), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n_rows);
    return hipGetLastError();
}

hipError_t launch_narrow16(const void* src, void* dst, int64_t n_rows, hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(narrow16_kernel, dim3((unsigned)((n_rows * 2 + 255) / 256)), dim3(256), 0, s, (const uint4*)src, (uint4*)dst, n_rows);
    return hipGetLastError();
}

hipError_t launch_rt_limits(const Params& p, hipStream_t s) {
    const int64_t rows = max_query_rows(p);
    if (p.batch <= 0 || rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(rt_limits_kernel, dim3((unsigned)((rows + 255) / 256), 1, (unsigned)p.batch), dim3(256), 0, s, p);
    return hipGetLastError();
}

size_t schedule_bytes(int32_t batch) {
    return QUEUE_WORDS * sizeof(int32_t) + ((((size_t)batch * sizeof(int32_t)) + 255) & ~(size_t)255);
}

// Calls without the schedule's launch against with it, of 663 calls of all sizes forward and 463 backward: forward, users of (nearly)
// equal keys 0.96 of the time, three of 349 slower by more than 1 %, and tiles that all find a place at once 0.87 on full layers, 0.93
// on target layers; otherwise up to 1.4.  Backward, equal keys and rows and a key block's rows shared by waves (with four of them whatever
// the rows) 0.97; users of unlike lengths 1.05, up to 1.4.  (The other kernels of the backward take their work from the counters that
// the schedule clears; dealt out in turn instead: 1.00 to 1.10 with equal users, up to 1.7 with others.)
static bool even_keys(const Params& p) { return mean_keys(p) >= 0.95 * (double)max_lead_keys(p); }
bool forward_needs_schedule(const Params& p) {
    if (p.rt_len) return true;  // the rows' limits
    const RowMap map = row_map(fwd_workgroup_rows(p), p.Hq, p.Hkv, max_query_rows(p));
    return !even_keys(p) && (int64_t)p.batch * p.Hkv * map.n_chunks * map.n_tiles > 512;
}
bool backward_needs_schedule(const Params& p, bool onepass) {
    if (p.rt_len || onepass || !even_keys(p)) return true;
    const int ways = dkdv_brief_ways(p);
    return ways == 0 || (ways != 4 && mean_rows(p) < 0.9 * (double)max_query_rows(p));
}

hipError_t launch_schedule(const Params& p, void* region, hipStream_t s) {
    if (p.batch <= 0) return hipSuccess;
    int32_t* counters = (int32_t*)region;
    int32_t* order = schedule_order(region);
    const int64_t rank_groups = (p.batch + RANK_USERS - 1) / RANK_USERS;
    const int64_t limit_groups = p.rt_len ? (std::max<int64_t>(max_query_rows(p), 0) + RANK_THREADS - 1) / RANK_THREADS : 0;
    const bool together = p.batch <= RANK_SORT_MAX && rank_groups + limit_groups * p.batch < (1ll << 31);
    if (p.rt_len && !together) {
        const hipError_t e = launch_rt_limits(p, s);
        if (e != hipSuccess) return e;
    }
    if (p.batch <= RANK_SORT_MAX)
        hipLaunchKernelGGL(schedule_rank_kernel, dim3((unsigned)(rank_groups + (together ? limit_groups * p.batch : 0))), dim3(RANK_THREADS), 0, s,
                           p, counters, order, (unsigned)rank_groups, (unsigned)std::max<int64_t>(limit_groups, 1));
    else
        hipLaunchKernelGGL(schedule_bucket_kernel, dim3(1), dim3(SCHED_THREADS), 0, s, p, counters, order);
    return hipGetLastError();
}

}  // namespace hta
