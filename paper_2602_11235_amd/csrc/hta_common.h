// Internal declarations shared by the translation units of libmtfm_hta.so (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

namespace hta {

// Everything one call needs, passed to the kernels by value.
struct Params {
    const void* q;
    const void* k;
    const void* v;
    void* out;            // fwd: output; bwd: the saved forward output (read only)
    float* lse;           // [Hq][total_q]
    const void* dout;     // bwd only
    void* dq;
    void* dk;
    void* dv;
    const int32_t* q_off;   // [B+1]
    const int32_t* kv_off;  // [B+1]
    const int32_t* hist_len;
    const int32_t* n_targets;
    int32_t batch;
    int64_t total_q;
    int64_t total_kv;
    int32_t max_hist;
    int32_t max_targets;
    int32_t Hq;
    int32_t Hkv;
    int32_t d;
    float scale;
    int32_t layer;        // 0 full (queries = all tokens), 1 target (queries = target tokens)
    // carved out of the caller's workspace (bwd)
    float* neg_delta;     // [Hq][total_q]   -<dout_i, out_i>
    float* neg_lse_s;     // [Hq][total_q]   -lse_i / scale: what the S accumulators of the dK/dV pass start from
    const int32_t* order; // [batch] users by decreasing tile count (bf16 path), or null = identity
    int32_t* queue;       // [N_XCD] work counters of the kernel being launched (bf16 path), zero when it starts
    // real-time tokens (mask rule 2); all null / 0 for samples of history + target tokens only
    const int32_t* rt_len;  // [B] real-time tokens of each user, between its history and its target tokens
    const int32_t* ts;      // [total_kv] one timestamp per K/V row
    int32_t max_rt;
    // the pointwise reading of phi2: weights norm * silu(scale s) instead of a row softmax (no lse, no delta)
    int32_t pointwise;
    float norm;
    // forward pass of a few requests (hta_serve_bf16.hip): workgroups an item's keys are split over; 0 = the ordinary kernel
    int32_t n_splits;
    float* o_part;          // [n_splits][total_q][Hq][d] partial outputs, each normalised by its own sum
    float* lse_part;        // [n_splits][Hq][total_q]    logsumexp of each split's keys (-inf: the row sees none; a mark: the user has fewer splits)
    int32_t* lim;           // [total_q] carved out of the workspace: number of leading K/V rows of the user (history, then
                            // the real-time tokens strictly earlier than the query) that the query row sees
};

// number of query rows a user can have at most, from the host-known bounds
__host__ __device__ inline int64_t max_query_rows(const Params& p) {
    return p.layer == 0 ? (int64_t)p.max_hist + p.max_rt + p.max_targets : (int64_t)p.max_targets;
}
// number of keys a user's tile loops can reach at most: history, then real-time tokens
__host__ __device__ inline int64_t max_lead_keys(const Params& p) { return (int64_t)p.max_hist + p.max_rt; }
// What the host knows of a call's average user, for the rules that choose a kernel: query rows, and keys of the tile loops
// (a full layer's totals do not tell its target tokens apart; half of the bound is as good a guess as any).
inline double mean_rows(const Params& p) { return (double)p.total_q / p.batch; }
inline double mean_keys(const Params& p) {
    const double keys = p.layer == 0 ? mean_rows(p) - 0.5 * p.max_targets : (double)(p.total_kv - p.total_q) / p.batch;
    return keys < 1. ? 1. : keys > (double)max_lead_keys(p) ? (double)max_lead_keys(p) : keys;
}
// The most keys that a user can have: the bound, and no more than all users have together.
inline int64_t most_keys(const Params& p) {
    const int64_t all = p.layer == 0 ? p.total_kv : p.total_kv - p.total_q, bound = max_lead_keys(p);
    return all < bound ? all : bound;
}
// What the longest user is taken to have where a form is chosen: the bounds of a call (of a captured graph, say) may be far above its lengths, which
// looks like a few long users among many short ones, and is the likelier where the bound is above two and a half times the mean.  (Requests
// with bounds of four and eight times their longest: by the bound the chosen form takes 1.065 of the best one's time, by this 1.025; with
// histories of a heavy tail and true bounds 1.007 and 1.009.)
inline double longest_keys(const Params& p) { return std::min((double)most_keys(p), 2.5 * mean_keys(p)); }
// Mask rule 2 (Section 3.2.2): a real-time token is visible only to tokens with later timestamps.  The real-time
// segment of a user is sorted by time, so the real-time keys a query sees are a prefix of it: those strictly earlier
// than the query.  lim[row] = hist_len + that prefix length = the number of leading K/V rows of the user the row
// attends to in the tile loops (its own key, when it is a real-time or target token, is a separate term).
__device__ inline void rt_limit_of_row(const Params& p, int b, int row) {
    const int L = p.hist_len[b], R = p.rt_len[b], T = p.n_targets[b];
    const int n_rows = p.layer == 0 ? L + R + T : T;
    if (row >= n_rows) return;
    const int32_t* ts = p.ts + p.kv_off[b];
    const int32_t t = ts[p.layer == 0 ? row : L + R + row];
    int lo = 0, hi = R;  // first real-time token that is not strictly earlier than t
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ts[L + mid] < t) lo = mid + 1; else hi = mid;
    }
    p.lim[(int64_t)p.q_off[b] + row] = L + lo;
}
// Where a query row's S and dP start from in the dK/dV passes: the address of -lse/scale (lanes of the wave's lower half) or
// of -delta (upper half), element idx = head * total_q + row.  A lane that stands for no row (not live) repeats the Q and dO of a row
// of its own user and names that one: its S starts from the sentinel behind the -lse/scale array, so its weight is exactly 0,
// but 0 times its dP still enters dK, and that must not carry another user's inf or NaN.
__device__ inline const float* row_start(const Params& p, int half, int64_t idx, bool live) {
    return half == 0 ? p.neg_lse_s + (live ? idx : (int64_t)p.Hq * p.total_q) : p.neg_delta + idx;
}
// the limits of all rows in a launch of their own (launch_schedule finds them otherwise)
hipError_t launch_rt_limits(const Params& p, hipStream_t s);

hipError_t launch_fwd_fp32(const Params& p, hipStream_t s);
hipError_t launch_bwd_fp32(const Params& p, hipStream_t s);
hipError_t launch_fwd_bf16(const Params& p, hipStream_t s);
hipError_t launch_serve_bf16(const Params& p, hipStream_t s);
hipError_t launch_bwd_bf16(const Params& p, hipStream_t s);
bool bwd_is_onepass(const Params& p);                           // one kernel for dQ, dK, dV: hta_bwd_onepass_bf16.hip
double onepass_us(const Params& p);                             // its estimated time, infinite where it does not fit
bool onepass_asks_late(const Params& p);                        // does it take its next items late in the current ones?
hipError_t launch_bwd_onepass_bf16(const Params& p, hipStream_t s);
bool bwd_is_brief(const Params& p);                             // little work: the kernels of hta_bwd_brief_bf16.hip, no schedule
hipError_t launch_bwd_brief_bf16(const Params& p, hipStream_t s);
int bwd_brief_ways(const Params& p, bool* dq_first);            // waves per key block there, and whether dQ's workgroups come first
int dkdv_brief_ways(const Params& p);                           // ... > 0: their dK/dV part behind the ordinary dQ pass
bool dkdv_is_resident(const Params& p);                         // the ordinary dK/dV pass would keep each user's rows in LDS
int dkdv_list_spread(const Params& p);                          // ... or not: its key tiles of a user are dealt to 2^this lists
hipError_t launch_dkdv_brief_bf16(const Params& p, hipStream_t s);
// the two launches of launch_bwd_bf16 that live in translation units of their own (other compiler options)
hipError_t launch_bwd_dq_bf16(const Params& p, hipStream_t s);       // dQ and the self-key blocks, every head_dim
hipError_t launch_bwd_dkdv128_bf16(const Params& p, hipStream_t s);  // dK/dV at head_dim 128, softmax weights
bool bf16_supported(int32_t d, int32_t Hq, int32_t Hkv);
// bf16 rows of 16 features <-> rows of 32 with a zero upper half ([n_rows][16] and [n_rows][32], 16-byte aligned): how
// head_dim 16 rides the 32-wide matrix tiles
constexpr int32_t BF16_PADDED_FROM = 16, BF16_PADDED_TO = 32;
hipError_t launch_widen16(const void* src, void* dst, int64_t n_rows, hipStream_t s);
hipError_t launch_narrow16(const void* src, void* dst, int64_t n_rows, hipStream_t s);
// the most key splits the bf16 forward pass may use for these host-known bounds: what its workspace has room for (1 = none)
int fwd_key_splits(int32_t batch, int32_t Hq, int32_t Hkv, int32_t d, int64_t max_rows, int64_t max_keys);
// the splits it does use, at most `room`; 0: the call runs the ordinary forward kernel
int serve_splits(const Params& p, int room);
// blocks of 32 rows per workgroup of the kernel for a few requests, once p.n_splits is set
int serve_row_blocks(const Params& p);
// ... and whether its work stands in a list or in a grid
bool serve_takes_list(const Params& p);
// packed (row, head) pairs that a workgroup of the ordinary forward kernel takes in this call
int fwd_workgroup_rows(const Params& p);
// stores the calling thread's error message (what mtfm_hta_last_error() returns) and hands `code` back
int report_error(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
// event hooks around each kernel (no-ops unless timing was enabled through the C ABI); `kind` is one of the
// MTFM_HTA_KERNEL_* values
void timing_begin(int kind, hipStream_t s);
void timing_end(int kind, hipStream_t s);
// The schedule region at the head of the workspace: work counters (one per kernel kind and XCD, 256 bytes in all),
// then the user order of the launch, long histories first.  launch_schedule() zeroes the former, builds the latter
// and, in calls with real-time tokens, fills p.lim.
constexpr int N_XCD = 8;
constexpr int QUEUE_DKDV = 0;  // kernel kinds that take their work from counters
constexpr int QUEUE_WORDS = 64;
size_t schedule_bytes(int32_t batch);
// Does it pay for its launch?  (p.order and p.queue stay null otherwise: users in the order given, kernels without a queue.)
bool forward_needs_schedule(const Params& p);
bool backward_needs_schedule(const Params& p, bool onepass);
hipError_t launch_schedule(const Params& p, void* region, hipStream_t s);
inline int32_t* schedule_order(void* region) { return (int32_t*)region + QUEUE_WORDS; }
inline int32_t* schedule_queue(void* region, int kind) { return (int32_t*)region + kind * N_XCD; }
__device__ inline int scheduled_user(const Params& p, int slot) { return p.order ? p.order[slot] : slot; }
// Placement of workgroups.  Work is a list of groups (user slot, y) -- y = kv head (x head chunk) -- each with up
// to `tpg` tiles that share operands (the K/V of the group, or its Q/dO).  The chip has 8 XCDs, each with its own
// L2, and hands consecutive workgroup ids to them round-robin; so id -> (xcd = id % 8, slot = id / 8), a group lives
// on one XCD (its tiles are consecutive slots there, so they also run close in time), and groups are dealt to the
// XCDs round-robin in schedule order, which keeps the long-first order inside every XCD.  Only locality depends
// on the round-robin assumption, never correctness.
struct WorkItem {
    int user_slot, y, tile;
    bool valid;
};
__device__ inline WorkItem decode_work(unsigned id, int n_groups, int ny, int tpg) {
    const int xcd = id % N_XCD, slot = id / N_XCD;
    const int gl = slot / tpg;
    const int group = gl * N_XCD + xcd;
    WorkItem w;
    w.valid = group < n_groups;
    w.tile = slot - gl * tpg;
    w.user_slot = group / ny;
    w.y = group - w.user_slot * ny;
    return w;
}
// The same where groups may be few, or few of them long: the tiles of a group are dealt to 2^spread XCDs in turn.  For grids, which do not
// balance themselves over the XCDs (17 users of which one has half of the work, two kv heads: that half ran on two XCDs), and for lists that
// the work counters below serve, where an XCD works off its own list first (list_spread).
__device__ inline WorkItem decode_spread(unsigned id, int n_groups, int ny, int tpg, int spread) {
    WorkItem w = decode_work(id, n_groups << spread, ny << spread, (tpg + (1 << spread) - 1) >> spread);
    w.tile = (w.tile << spread) + (w.y & ((1 << spread) - 1));
    w.y >>= spread;
    return w;
}
// Spread of a training launch: at least 128 shares of groups for the 8 XCDs, 512 where the longest user has more than twice the
// mean's rows (that case of 17 users 2.22 -> 1.02 ms per step, 16 users of 630..2420 keys 0.60 -> 0.47; 93 users of up to 8192
// keys 4.74 -> 4.61 ms).  Tiles of a group on more XCDs read its operands into more L2s: with four shares of every one of 512
// equal groups a step was 6 % slower.
inline int grid_spread(const Params& p, int64_t n_groups, int64_t tpg) {
    const int64_t shares = n_groups >= 128 && (double)max_query_rows(p) * p.batch > 2. * p.total_q ? 512 : 128;
    int s = 0;
    while (s < 3 && (n_groups << s) < shares && (2 << s) <= tpg) s++;
    return s;
}
inline int64_t work_grid(int64_t n_groups, int64_t tpg, int spread = 0) {
    return (((n_groups << spread) + N_XCD - 1) / N_XCD) * N_XCD * ((tpg + (1 << spread) - 1) >> spread);
}

// Work distribution for kernels with long work items (the dK/dV pass: tens of microseconds per item).  The hardware
// hands the workgroups of a grid to the shader engines in a fixed rotation, whatever each has left to do, so with items
// of unequal length (jagged users) whole compute units run dry while others queue up: a fifth of the chip on the
// paper's length mix.  Such a kernel launches only as many workgroups as the chip holds at once, and each takes work
// item after work item from a counter (kernels with short items lose more to the hand-over than they gain): XCD x
// serves the ids x, x + 8, x + 16, ... (a group's tiles on one L2, as above, or on those of a spread group), in order, through counters[x];
// a workgroup whose own XCD has nothing left helps the others.  The loop ends for a workgroup once every counter has
// passed the end of its list, which every workgroup reaches.
// The first round needs no counter: a workgroup's index is its first id, and the counters count what is taken behind that.
// A list that is exhausted is read and not counted up: the counters share a cache line, whose atomics come one after the other, and 512
// workgroups that tried all eight lists before they left took 45 us to leave.  (The one-pass backward, where calls of few items paid
// for it: 63 users of a full layer, 103 keys, 16/4 heads, 51.9 -> 31.9 us, 254 users x 570 keys x 47, 8/2 heads, 96.2 -> 62.5, 0.96 of
// the time on average over 1815 sampled calls that take it.  The streaming dK/dV pass of a small call: whole backward of 150 users of
// 328 keys, 4/4 heads, 171 -> 132 us.)
//   ids of XCD x's list that the first round deals out, n_groups workgroups in all
__device__ inline unsigned queue_dealt(unsigned n_groups, int x) { return (n_groups + N_XCD - 1 - (unsigned)x) / N_XCD; }
//   thread 0:  take the next slot of the own XCD shortly before an item ends ...  (An atomic on an address that the compiler can prove uniform becomes a
//   reduction over the wave, which reads the result back at once: wave 0 waits for it here, and for what it has in flight.)
__device__ inline unsigned queue_take_ahead(int32_t* counters, int xcd, unsigned per_xcd, unsigned n_groups) {
    const unsigned dealt = queue_dealt(n_groups, xcd);
    return dealt < per_xcd ? dealt + atomicAdd((unsigned*)&counters[xcd], 1u) : per_xcd;
}
//   or, in two steps, ask for it: `answer` gets a count behind the dealt ones, and nothing waits for the atomic ...
__device__ inline void queue_ask(unsigned& answer, int32_t* counters, int xcd, unsigned per_xcd, unsigned n_groups) {
    if (queue_dealt(n_groups, xcd) >= per_xcd) return;
    int x = xcd;
    asm volatile("" : "+v"(x));
    answer = atomicAdd((unsigned*)&counters[x], 1u);
}
//   ... before the answer is read, which all lanes of the first wave do, in front of the item's results (whose stores would be waited for with it)
__device__ inline unsigned queue_answer(unsigned answer, int xcd, unsigned per_xcd, unsigned n_groups) {
    const unsigned dealt = queue_dealt(n_groups, xcd);
    return dealt < per_xcd ? __builtin_amdgcn_readfirstlane(answer) + dealt : per_xcd;
}
//   first wave:  ... and turn it into a work id, or -1 when all lists are exhausted.  (Lane q looks at the list of XCD xcd + q: one
//   load, and none of the addresses is kept in registers for the length of every item.)
__device__ inline int queue_resolve(int32_t* counters, int xcd, unsigned taken, unsigned per_xcd, unsigned n_groups) {
    taken = __builtin_amdgcn_readfirstlane(taken);
    if (taken < per_xcd) return (int)(taken * N_XCD + xcd);
    if (n_groups >= per_xcd * N_XCD) return -1;  // the first round was all
    int lane;  // (anew, for the same reason)
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    const int x = (xcd + lane) % N_XCD;
    bool left = false;  // (a list only ever shortens: one that is seen exhausted is, one that is not may be by now)
    if (lane > 0 && lane < N_XCD)
        left = queue_dealt(n_groups, x) + __hip_atomic_load((unsigned*)&counters[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < per_xcd;
    for (uint64_t lists = __builtin_amdgcn_ballot_w64(left); lists != 0; lists &= lists - 1) {
        const int from = (xcd + __builtin_ctzll(lists)) % N_XCD;
        unsigned slot = 0;
        if (lane == 0) slot = queue_dealt(n_groups, from) + atomicAdd((unsigned*)&counters[from], 1u);
        slot = __builtin_amdgcn_readfirstlane(slot);
        if (slot < per_xcd) return (int)(slot * N_XCD + from);
    }
    return -1;
}
// workgroups of `Kernel` (at `threads` threads, no dynamic LDS) that the current device holds at once
template <auto Kernel>
inline int resident_workgroups(int threads) {
    constexpr int MAX_DEVICES = 64;
    static std::atomic<int> cached[MAX_DEVICES];  // per device (0: not asked yet); the answer never changes
    int dev = 0, n_cu = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    const bool cacheable = dev >= 0 && dev < MAX_DEVICES;
    if (cacheable) {
        const int known = cached[dev].load(std::memory_order_relaxed);
        if (known > 0) return known;
    }
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, Kernel, threads, 0) != hipSuccess) return 256;
    const int n = n_cu * (per_cu > 0 ? per_cu : 1);
    if (cacheable) cached[dev].store(n, std::memory_order_relaxed);
    return n;
}
// fill `n` 32-bit words with zero (a kernel, so that a caller may capture the call in a HIP graph)
hipError_t launch_zero_words(void* ptr, size_t n_words, hipStream_t s);

}  // namespace hta
