// Fused group layer normalization (Section 3.2.2, the fused operator of Section 3.3.2) for gfx950: forward,
// backward and the C ABI of include/mtfm_gln.h.
//
// The work is bound by HBM: a token is read once and written once, its arithmetic is a few dozen flops per
// element.  One wave owns a token at a time: lane l holds features [8 l, 8 l + 8) of every 512-feature chunk
// (16-byte loads of bf16), the two row statistics are wave reductions in registers, and nothing is gathered or
// scattered -- a token picks its group's parameter row out of LDS, where all rows are staged once per workgroup.
// Tokens of at most 256 (128) features take half (a quarter) of a wave, two (four) of them side by side.
// Workgroups are persistent (a fixed grid strides over the tokens), which also bounds the number of partial
// parameter gradients of the backward pass: each workgroup accumulates dgamma / dbeta of all groups in LDS
// and writes its share once; a second kernel sums the shares.  All sums are in a fixed order.
// us of a call, among others, bf16, as (tokens x features, groups), the kernels with a wave per token and LDS atomics -> these:
//   forward   gated 200 000 x 136, 8  82.8 -> 37.7   200 000 x 256, 8  87.9 -> 55.4   200 000 x 512, 8  110.2 -> 108.0
//             plain 130 000 x 640, 2  83.2 -> 67.3   200 000 x 1024, 8  153.0 -> 148.1
//   backward  gated   9 418 x 688, 5  63.4 -> 24.1    18 374 x 1008, 4  93.6 -> 48.3   200 000 x 512, 8  229.1 -> 216.5 (4.7 TB/s)
//             gated  20 000 x 136, 8  24.9 -> 15.7   200 000 x 1024, 8  459.8 -> 418.0   plain 11 837 x 928, 4  68.0 -> 23.8
#include "../../include/mtfm_gln.h"
#include "hta_common.h"

#include <hip/hip_runtime.h>

namespace gln {

constexpr int THREADS = 512;
constexpr int WAVES = THREADS / 64;
constexpr int MAX_BLOCKS = 512;   // workgroups of a forward launch
constexpr int MAX_SHARES = 256;   // workgroups of a backward launch: one per compute unit (two of half the size: twice the shares to write and sum)
constexpr int WORKSPACE_SHARES = 512;  // shares of dgamma / dbeta that the workspace has room for: what callers were asked for when the grid was twice this, and are still
constexpr int CHUNK = 512;        // features a wave covers per pass: 64 lanes x 8
constexpr int MAX_CHUNKS = 4;     // d_model <= 2048
constexpr int MAX_TABLE = 8192;   // n_groups x padded row length, in floats
constexpr int MAX_GROUPS = MAX_TABLE / CHUNK;
constexpr int REDUCE_THREADS = 512, REDUCE_WAVES = REDUCE_THREADS / 64, REDUCE_COLS = 32, REDUCE_SLICES = REDUCE_THREADS / (REDUCE_COLS / 4);
static_assert(MAX_SHARES % REDUCE_SLICES == 0, "a lane's shares");

constexpr int LDS_FLOATS = 32768;  // of the backward kernel's parameter rows and accumulators (the rest of the 160 KB: its sort)
static_assert(2 * MAX_TABLE <= LDS_FLOATS, "the forward kernel's parameter rows");
static_assert((LDS_FLOATS + 1024 + MAX_GROUPS * 16) * sizeof(float) <= 160 * 1024, "the backward kernel's, with 16 waves");
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct Args {
    const void *x, *gate, *dy;
    const int32_t* group_id;
    const float *gamma, *beta, *mean_in, *rstd_in;
    void *y, *dx, *dgate;
    float *mean, *rstd, *partials;
    int64_t n;
    int32_t d, n_groups, row;  // row = d rounded up to what a token's lanes hold: the stride of a group's row in LDS
    int32_t span;              // backward: tokens a wave takes per pass, at most 64
    int32_t rep;               // backward: copies of the accumulators in LDS
    float eps;
};

// Backward: threads of a workgroup, one per compute unit with as many waves as the registers of a token's chunks and sums allow without scratch
// (which costs a small call 4 to 10 us by itself), and sets of tokens that a wave has in flight.  Two chunks in bf16, eight waves with two tokens
// in flight against twelve with one or sixteen with one and scratch: 60 000 x 736, 8 groups, gated 104 / 104 / 112 us, 9418 x 688 24.2 / 24.8 / 33.7.
// (Four chunks in float32 with a gate keep 12 registers in scratch; four waves without against these eight: 64 x 2048 13.2 against 15.1 us,
// 1000 x 1544 21.3 against 20.1, 20 000 x 2048 183 against 185, 60 000 x 1544 411 against 410; the other kinds of four chunks lose by four waves.)
constexpr int bwd_threads(int CPL) { return CPL == 1 ? 1024 : 512; }
template <typename T, int CPL, int LPT, bool GATED>
constexpr int bwd_depth() { return sizeof(T) == 2 && (CPL == 2 || (CPL == 1 && (LPT == 64 || !GATED))) ? 2 : 1; }
// Calls of few tokens that lie side by side in a wave: half as many waves, and a token to each while there are compute units left.  Such a call is the
// latency of one workgroup and of the sum of its shares, and tokens of other groups in the same wave come one after the other: sixteen waves and side
// by side from the first token on, us of a call among others (9 of them the host's), gated, 4 groups: 64 x 64 11.8 -> 9.2, 2000 x 64 12.0 -> 9.1,
// 2000 x 128 12.1 -> 9.5, 16 groups 16.1 -> 11.8; 8000 x 136 12.0 -> 11.5.  With more than two sets of tokens to each of 2048 waves sixteen waves are
// as fast or faster: 32 000 x 128 16.3 against 16.1, 16 000 x 256 15.6 against 16.0, 32 000 x 136 18.8 against 21.0.
constexpr int BRIEF_THREADS = 512;
bool is_brief(int64_t n, int lanes_per_token) { return lanes_per_token < 64 && n <= (int64_t)2 * (64 / lanes_per_token) * MAX_SHARES * (BRIEF_THREADS / 64); }

// eight consecutive features as they lie in memory; converted where they are used, so that tokens waiting for
// their turn occupy half the registers in bf16
template <typename T>
struct Raw;
template <>
struct Raw<__bf16> {
    bf16x8 v;
    __device__ void load(const __bf16* p) { v = __builtin_nontemporal_load((const bf16x8*)p); }
    __device__ float operator[](int j) const { return (float)v[j]; }
    __device__ void forget() { asm volatile("" : "+v"(v)); }  // what follows is formed from these registers again, not kept from before
};
template <>
struct Raw<float> {
    floatx4 lo, hi;
    __device__ void load(const float* p) { lo = *(const floatx4*)p, hi = *(const floatx4*)(p + 4); }
    __device__ float operator[](int j) const { return j < 4 ? lo[j] : hi[j - 4]; }
    __device__ void forget() { asm volatile("" : "+v"(lo), "+v"(hi)); }
};

__device__ inline void store8(__bf16* p, const float (&f)[8]) {
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; j++) v[j] = (__bf16)f[j];  // round to nearest even
    __builtin_nontemporal_store(v, (bf16x8*)p);  // written once, not read again by this kernel
}
__device__ inline void store8(float* p, const float (&f)[8]) {
    floatx4 a, b;
#pragma unroll
    for (int j = 0; j < 4; j++) a[j] = f[j], b[j] = f[4 + j];
    *(floatx4*)p = a;
    *(floatx4*)(p + 4) = b;
}

template <int CTRL>
__device__ inline float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
// Sum over the LPT lanes of a token, the same value in all of them, in a fixed order: exchanges inside the 16-lane rows (lane ^ 1, lane ^ 2,
// mirror of each half row, mirror of the row), then the sums of the token's rows.
template <int LPT>
__device__ inline float token_sum(float v) {
    v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp<0x141>(v);  // row_half_mirror
    v += dpp<0x140>(v);  // row_mirror
    if constexpr (LPT == 16) return v;
    const int u = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(u, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(u, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(u, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(u, 48));
    if constexpr (LPT == 32) return (threadIdx.x & 32) ? r2 + r3 : r0 + r1;
    return (r0 + r1) + (r2 + r3);
}

// Where feature e of a parameter or accumulator row lies in LDS, for chunks of CH features.  A lane reads its 8 features of a chunk as
// two 16-byte words: the first words of a token's lanes are contiguous, then the second words, so neither read has a bank conflict.
template <int CH>
__device__ inline int quad_slot(int e) {
    const int r = e & (CH - 1);
    return (e - r) + ((r >> 2) & 1) * (CH / 2) + (r >> 3) * 4 + (r & 3);
}

template <int CH, int NTHR>
__device__ inline void stage_rows(float* table, const float* src, int n_groups, int d, int row) {
    const int quads = d / 4;
    for (int i = threadIdx.x; i < n_groups * quads; i += NTHR) {
        const int g = i / quads, e = (i - g * quads) * 4;
        *(floatx4*)&table[g * row + quad_slot<CH>(e)] = *(const floatx4*)&src[i * 4];
    }
}

template <int LPT>
__device__ inline void read_row8(const float* table_row, int c, int fl, float (&f)[8]) {
    const floatx4 a = *(const floatx4*)&table_row[c * LPT * 8 + fl * 4];
    const floatx4 b = *(const floatx4*)&table_row[c * LPT * 8 + LPT * 4 + fl * 4];
#pragma unroll
    for (int j = 0; j < 4; j++) f[j] = a[j], f[4 + j] = b[j];
}

__device__ inline int clamp_group(int g, int n_groups) { return g < 0 ? 0 : (g >= n_groups ? n_groups - 1 : g); }

// LPT lanes hold a token (64 of 512 features and CPL such chunks, 32 of at most 256 features, 16 of at most 128); 64 / LPT tokens lie side by
// side in a wave, and TPW such sets are in flight: their loads are all issued before the first is used, those of the first iteration before the
// parameters are staged and, where tokens lie side by side (200 000 x 136: 45 -> 37.7 us), those of the next while the current one is worked on.
template <typename T, int CPL, int LPT, bool GATED>
__global__ __launch_bounds__(THREADS, CPL <= 2 ? 4 : 2) void fwd_kernel(const Args a) {
    constexpr int TPW = CPL == 1 ? 2 : 1, NT = 64 / LPT, CH = LPT * 8;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* gamma_s = smem;
    float* beta_s = smem + a.n_groups * a.row;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, fl = lane % LPT, sub = lane / LPT;
    const int d = a.d;
    const float inv_d = 1.f / (float)d;
    const T* xg = (const T*)a.x;
    const T* ug = (const T*)a.gate;
    T* yg = (T*)a.y;
    Raw<T> xr[TPW][CPL], ur[TPW][CPL];
    int gr[TPW];
    const auto fetch = [&](int64_t t0, bool ids) {
#pragma unroll
        for (int k = 0; k < TPW; k++) {
            const int64_t t = t0 + k * NT + (NT > 1 ? sub : 0);
            if (ids) gr[k] = t < a.n ? a.group_id[t] : 0;
#pragma unroll
            for (int c = 0; c < CPL; c++)
                if (t < a.n && (c * LPT + fl) * 8 < d) xr[k][c].load(xg + t * d + (c * LPT + fl) * 8);
#pragma unroll
            for (int c = 0; c < CPL; c++)
                if (GATED && t < a.n && (c * LPT + fl) * 8 < d) ur[k][c].load(ug + t * d + (c * LPT + fl) * 8);
        }
    };
    const auto work = [&](int64_t t0, const Raw<T> (&xs)[TPW][CPL], const Raw<T> (&us)[TPW][CPL], const int (&gs)[TPW], bool late) {
#pragma unroll
        for (int k = 0; k < TPW; k++) {
            const int64_t t = t0 + k * NT + (NT > 1 ? sub : 0);
            if (NT == 1 && t >= a.n) break;
            float xv[CPL][8], s = 0.f;
#pragma unroll
            for (int c = 0; c < CPL; c++)
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    xv[c][j] = t < a.n && (c * LPT + fl) * 8 < d ? xs[k][c][j] : 0.f;
                    s += xv[c][j];
                }
            // Centre on a first mean m, then correct it by the mean of the centred values: x - m is exact for a
            // token whose spread is small against its offset, where the rounding of m itself would dominate.
            const float m = token_sum<LPT>(s) * inv_d;
            float q = 0.f, r = 0.f;
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                if ((c * LPT + fl) * 8 < d) {
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        xv[c][j] -= m;
                        r += xv[c][j];
                        q += xv[c][j] * xv[c][j];
                    }
                }
            }
            const float delta = token_sum<LPT>(r) * inv_d;
            const float var = fmaxf(token_sum<LPT>(q) * inv_d - delta * delta, 0.f);
            const float mean = m + delta;
            const float rstd = 1.f / sqrtf(var + a.eps);
            if (NT > 1 && t >= a.n) break;  // (behind the sums: lanes of the same token leave together)
            const int id = late ? a.group_id[t] : gs[k];
            const int g = clamp_group(NT == 1 ? __builtin_amdgcn_readfirstlane(id) : id, a.n_groups);
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                const int col = (c * LPT + fl) * 8;
                if (col < d) {
                    float gm[8], bt[8], out[8];
                    read_row8<LPT>(gamma_s + g * a.row, c, fl, gm);
                    read_row8<LPT>(beta_s + g * a.row, c, fl, bt);
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        out[j] = gm[j] * ((xv[c][j] - delta) * rstd) + bt[j];
                        if (GATED) out[j] *= us[k][c][j];
                    }
                    store8(yg + t * d + col, out);
                }
            }
            if (fl == 0) {
                if (a.mean) a.mean[t] = mean;
                if (a.rstd) a.rstd[t] = rstd;
            }
        }
    };
    const int64_t stride = (int64_t)gridDim.x * WAVES * TPW * NT;
    int64_t t0 = ((int64_t)blockIdx.x * WAVES + wave) * (TPW * NT);
    fetch(t0, true);
    stage_rows<CH, THREADS>(gamma_s, a.gamma, a.n_groups, d, a.row);
    stage_rows<CH, THREADS>(beta_s, a.beta, a.n_groups, d, a.row);
    __syncthreads();
    if constexpr (NT > 1) {
        for (; t0 < a.n; t0 += stride) {
            Raw<T> xs[TPW][CPL], us[TPW][CPL];
            int gs[TPW];
#pragma unroll
            for (int k = 0; k < TPW; k++) {
                gs[k] = gr[k];
#pragma unroll
                for (int c = 0; c < CPL; c++) xs[k][c] = xr[k][c], us[k][c] = ur[k][c];
            }
            if (t0 + stride < a.n) fetch(t0 + stride, true);
            work(t0, xs, us, gs, false);
        }
    } else {
        // (no further ahead: two workgroups per compute unit have enough in flight.  Two chunks and a gate: the id is asked for behind the sums;
        // with the loads, 200 000 x 1024 took 233 us in place of 216, without a gate 148 in place of 152.)
        if (t0 < a.n) work(t0, xr, ur, gr, false);
        for (t0 += stride; t0 < a.n; t0 += stride) {
            fetch(t0, !(CPL > 1 && GATED));
            work(t0, xr, ur, gr, CPL > 1 && GATED);
        }
    }
}

// Backward.  A workgroup takes a span of up to 64 consecutive tokens per wave and orders it by group (a counting sort of the ids in LDS);
// each wave then takes an equal share of the ordered span (lane l holds the group and position of its l-th token) and works
// through it group by group: the tokens of one group add their dz (.) xhat and dz into registers, which go to the workgroup's accumulators in
// LDS when the group is done.  A wave adds there without atomics: a group that ends inside its share is nobody else's to end, and the last group of
// its share, which the next waves may go on with, waits until all waves are through; then the waves of one group take turns, `rep` of
// them at a time in copies of the accumulators of their own.  (LDS float atomics run at a lane per clock: with them the flushes of 1.6 groups per
// wave took 30 to 45 us of a call, whatever its size.)
template <typename T, int CPL, int LPT, bool GATED, int NTHR>
__global__ __launch_bounds__(NTHR) void bwd_kernel(const Args a) {
    constexpr int NW = NTHR / 64, NT = 64 / LPT, CH = LPT * 8;
    constexpr int DEPTH = bwd_depth<T, CPL, LPT, GATED>();
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int table = a.n_groups * a.row;
    float* gamma_s = smem;
    float* beta_s = smem + table;                   // present only with a gate
    float* acc_s = smem + (GATED ? 2 : 1) * table;  // rep x [dgamma | dbeta]
    __shared__ int sorted_s[NTHR];                                        // (group << 16) | offset of the token in the span
    __shared__ __attribute__((aligned(16))) int counts_s[MAX_GROUPS * NW];  // tokens of each group among a wave's 64 candidates
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, fl = lane % LPT, sub = lane / LPT;
    const int d = a.d;
    const float inv_d = 1.f / (float)d;
    const T* dyg = (const T*)a.dy;
    const T* xg = (const T*)a.x;
    const T* ug = (const T*)a.gate;
    T* dxg = (T*)a.dx;
    T* dug = (T*)a.dgate;
    const int block_span = a.span * NW;
    int64_t base = (int64_t)blockIdx.x * block_span;
    int g_me = -1;
    if (base < a.n && (int)threadIdx.x < (int)min((int64_t)block_span, a.n - base)) g_me = a.group_id[base + threadIdx.x];
    stage_rows<CH, NTHR>(gamma_s, a.gamma, a.n_groups, d, a.row);
    if (GATED) stage_rows<CH, NTHR>(beta_s, a.beta, a.n_groups, d, a.row);
    for (int i = threadIdx.x * 4; i < 2 * a.rep * table; i += NTHR * 4) *(floatx4*)&acc_s[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int i = a.n_groups * NW + threadIdx.x; i < MAX_GROUPS * NW; i += NTHR) counts_s[i] = 0;

    for (; base < a.n; base += (int64_t)gridDim.x * block_span) {
        const int live = (int)min((int64_t)block_span, a.n - base);
        if (base != (int64_t)blockIdx.x * block_span) g_me = (int)threadIdx.x < live ? a.group_id[base + threadIdx.x] : -1;
        const bool mine = (int)threadIdx.x < live;
        g_me = mine ? clamp_group(g_me, a.n_groups) : -1;
        int rank = 0;
        for (int g = 0; g < a.n_groups; g++) {
            const uint64_t m = __ballot(g_me == g);
            if (g_me == g) rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            if (lane == 0) counts_s[g * NW + wave] = __builtin_popcountll(m);
        }
        __syncthreads();
        {   // every wave sums up the counts, a few consecutive ones to a lane, and each lane fetches where its (group, wave) starts
            constexpr int PER = MAX_GROUPS * NW / 64;
            int c[PER], before = 0;
#pragma unroll
            for (int i = 0; i < PER; i++) c[i] = counts_s[lane * PER + i], before += c[i];
            const int own = before;
#pragma unroll
            for (int m = 1; m < 64; m *= 2) {
                const int up = __shfl_up(before, m);
                if (lane >= m) before += up;
            }
            before -= own;
            int start = before;
#pragma unroll
            for (int i = 0; i + 1 < PER; i++) start += i < wave % PER ? c[i] : 0;
            static_assert(NW % PER == 0, "a lane's counts are of one group");
            const int pos = __shfl(start, (max(g_me, 0) * NW + wave) / PER) + rank;
            if (mine) sorted_s[pos] = (g_me << 16) | (int)threadIdx.x;
        }
        __syncthreads();
        const int per_wave = (live + NW - 1) / NW;
        int g_lane = -1, off_lane = 0;
        if (lane < per_wave && wave * per_wave + lane < live) {
            const int e = sorted_s[wave * per_wave + lane];
            g_lane = e >> 16, off_lane = e & 0xFFFF;
        }
        // the last groups of the waves' shares, a lane to a wave: where a run of equal ones starts, and the longest run
        const bool there = lane < NW && lane * per_wave < live;
        const int last = there ? sorted_s[min((lane + 1) * per_wave, live) - 1] >> 16 : -1;
        const int last_before = __shfl_up(last, 1);
        const uint32_t goes_on = (uint32_t)__ballot(there && lane > 0 && last == last_before);
        const uint32_t starts = ~goes_on & ((2u << wave) - 1);
        const int turn = wave - (31 - __builtin_clz(starts));  // (wave 0 always starts a run)
        int longest = 1;
        for (uint32_t m = goes_on; m; m &= m << 1) longest++;

        float acc_g[CPL][8], acc_b[CPL][8];
        const auto add_to = [&](float* acc, int g) {  // this wave's sums to the accumulators
            if (NT > 1) {
#pragma unroll
                for (int m = LPT; m < 64; m *= 2)
#pragma unroll
                    for (int j = 0; j < 8; j++) acc_g[0][j] += __shfl_xor(acc_g[0][j], m), acc_b[0][j] += __shfl_xor(acc_b[0][j], m);
            }
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                if ((NT == 1 || sub == 0) && (c * LPT + fl) * 8 < d) {
#pragma unroll
                    for (int h = 0; h < 2; h++) {
                        floatx4* pg = (floatx4*)&acc[g * a.row + c * CH + h * (CH / 2) + fl * 4];
                        floatx4* pb = (floatx4*)&acc[table + g * a.row + c * CH + h * (CH / 2) + fl * 4];
                        floatx4 vg = *pg, vb = *pb;
#pragma unroll
                        for (int j = 0; j < 4; j++) vg[j] += acc_g[c][4 * h + j], vb[j] += acc_b[c][4 * h + j];
                        *pg = vg;
                        *pb = vb;
                    }
                }
            }
        };
        // The tokens in order, NT of one group at a time, DEPTH such sets in flight.
        float mean_lane = 0.f, rstd_lane = 0.f;
        if (g_lane >= 0) mean_lane = a.mean_in[base + off_lane], rstd_lane = a.rstd_in[base + off_lane];
        const T* dy0 = dyg + base * d;
        const T* x0 = xg + base * d;
        const T* u0 = ug + base * d;
        T* dx0 = dxg + base * d;
        T* du0 = dug + base * d;
        uint64_t todo = __ballot(g_lane >= 0), members = 0;
        int g_next = -1;
        Raw<T> gv[DEPTH][CPL], xv[DEPTH][CPL], uv[DEPTH][CPL];
        int group[DEPTH], index[DEPTH], offset[DEPTH];  // group: -1 behind the last set; offset: of the lane's token in the span, -1 for none
        const auto fetch = [&](int k) {
            if (!members) {
                g_next = todo ? __builtin_amdgcn_readlane(g_lane, __builtin_ctzll(todo)) : -1;
                members = todo ? __ballot(g_lane == g_next) : 0;
                todo &= ~members;
            }
            group[k] = g_next;
            if (g_next < 0) return;
            index[k] = 0, offset[k] = -1;
#pragma unroll
            for (int i = 0; i < NT; i++) {
                const int at = members ? __builtin_ctzll(members) : 0;
                const int off = members ? __builtin_amdgcn_readlane(off_lane, at) : -1;
                members &= members - 1;  // stays 0 once empty
                if (i == 0 || sub == i) index[k] = at, offset[k] = off;
            }
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                const int col = (c * LPT + fl) * 8;
                if ((NT == 1 || offset[k] >= 0) && col < d) {
                    gv[k][c].load(dy0 + offset[k] * d + col);
                    xv[k][c].load(x0 + offset[k] * d + col);
                    if (GATED) uv[k][c].load(u0 + offset[k] * d + col);
                }
            }
        };
#pragma unroll
        for (int k = 0; k < DEPTH; k++) fetch(k);
        int g = -1;  // the group that the sums in registers are of
        const auto work = [&](int k) {
            if (group[k] != g) {
                if (g >= 0) add_to(acc_s, g);
                g = group[k];
#pragma unroll
                for (int c = 0; c < CPL; c++)
#pragma unroll
                    for (int j = 0; j < 8; j++) acc_g[c][j] = 0.f, acc_b[c][j] = 0.f;
            }
            float mean, rstd;
            if constexpr (NT == 1) {
                mean = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mean_lane), index[k]));
                rstd = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, rstd_lane), index[k]));
            } else {
                mean = __shfl(mean_lane, index[k]), rstd = __shfl(rstd_lane, index[k]);
            }
            const bool there = NT == 1 || offset[k] >= 0;
            int fo = fl;
            asm volatile("" : "+v"(fo));  // (the group's parameters are read from LDS for each token: kept, they would be 32 registers)
            float s1 = 0.f, s2 = 0.f;
            float w[CPL][8];
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                const int col = (c * LPT + fl) * 8;
                if (there && col < d) {
                    float gm[8];
                    read_row8<LPT>(gamma_s + g * a.row, c, fo, gm);
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        const float xh = (xv[k][c][j] - mean) * rstd;
                        const float dz = GATED ? gv[k][c][j] * uv[k][c][j] : gv[k][c][j];
                        w[c][j] = dz * gm[j];
                        s1 += w[c][j];
                        s2 += w[c][j] * xh;
                        acc_g[c][j] += dz * xh;
                        acc_b[c][j] += dz;
                    }
                    if (GATED) {
                        float bt[8], du[8];
                        gv[k][c].forget();
                        xv[k][c].forget();
                        read_row8<LPT>(beta_s + g * a.row, c, fo, bt);
#pragma unroll
                        for (int j = 0; j < 8; j++) du[j] = gv[k][c][j] * (gm[j] * ((xv[k][c][j] - mean) * rstd) + bt[j]);
                        store8(du0 + offset[k] * d + col, du);
                    }
                }
                if (CPL > 1) __builtin_amdgcn_sched_barrier(0);  // (chunk by chunk: interleaved they want more than 128 registers)
            }
            s1 = token_sum<LPT>(s1) * inv_d;
            s2 = token_sum<LPT>(s2) * inv_d;
#pragma unroll
            for (int c = 0; c < CPL; c++) {
                const int col = (c * LPT + fl) * 8;
                if (there && col < d) {
                    float out[8];
                    xv[k][c].forget();
#pragma unroll
                    for (int j = 0; j < 8; j++) out[j] = rstd * (w[c][j] - s1 - (xv[k][c][j] - mean) * rstd * s2);
                    store8(dx0 + offset[k] * d + col, out);
                }
            }
        };
        for (bool more = group[0] >= 0; more;) {
#pragma unroll
            for (int k = 0; k < DEPTH; k++) {
                more = group[k] >= 0;
                if (!more) break;
                work(k);
                fetch(k);
            }
        }
        __syncthreads();
        for (int r = 0; r * a.rep < longest; r++) {
            if (r) __syncthreads();
            if (g >= 0 && turn / a.rep == r) add_to(acc_s + (turn % a.rep) * 2 * table, g);
        }
    }
    __syncthreads();
    // this workgroup's share, features in their natural order: [dgamma | dbeta][n_groups][d]
    const int gd = a.n_groups * d, quads = d / 4;
    float* share = a.partials + (size_t)blockIdx.x * 2 * gd;
    for (int i = threadIdx.x; i < 2 * a.n_groups * quads; i += NTHR) {
        const int g = i / quads, e = (i - g * quads) * 4;  // (rows of dgamma, then those of dbeta, as in LDS)
        floatx4 v = *(const floatx4*)&acc_s[g * a.row + quad_slot<CH>(e)];
        for (int r = 1; r < a.rep; r++) v += *(const floatx4*)&acc_s[r * 2 * table + g * a.row + quad_slot<CH>(e)];
        *(floatx4*)&share[i * 4] = v;
    }
}

// dgamma | dbeta = the sum of the workgroups' shares, in a fixed order: lane l of a wave takes columns 4 (l % 8) .. of the workgroup's
// and every 64th share, the eight lanes of a column add up, then the eight waves.  All latency, so every lane has its (at most
// four) loads of 16 bytes in flight at once and the columns are spread over the chip (256 shares of 2 x 8 x 512: 4.0 us).
__global__ __launch_bounds__(REDUCE_THREADS) void reduce_kernel(const float* partials, int n_shares, int gd, float* dgamma, float* dbeta) {
    __shared__ floatx4 part[REDUCE_WAVES][REDUCE_COLS / 4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quad = lane % (REDUCE_COLS / 4);
    const int first = blockIdx.x * REDUCE_COLS, e = first + 4 * quad;  // (gd is a multiple of 8: no quad has columns of both)
    const int slice = (int)threadIdx.x / (REDUCE_COLS / 4);
    const float* col4 = partials + min(e, 2 * gd - 4);  // (no branches: what is not there repeats what is, and does not count)
    floatx4 v[MAX_SHARES / REDUCE_SLICES];
#pragma unroll
    for (int i = 0; i < MAX_SHARES / REDUCE_SLICES; i++)
        v[i] = *(const floatx4*)(col4 + (size_t)max(0, min(i * REDUCE_SLICES + slice, n_shares - 1)) * 2 * gd);
    floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < MAX_SHARES / REDUCE_SLICES; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) s[j] += i * REDUCE_SLICES + slice < n_shares ? v[i][j] : 0.f;
#pragma unroll
    for (int m = REDUCE_COLS / 4; m < 64; m *= 2)
#pragma unroll
        for (int j = 0; j < 4; j++) s[j] += __shfl_xor(s[j], m);
    if (lane < REDUCE_COLS / 4) part[wave][quad] = s;
    __syncthreads();
    const int col = first + (int)threadIdx.x;
    if (threadIdx.x < REDUCE_COLS && col < 2 * gd) {
        float total = 0.f;
#pragma unroll
        for (int w = 0; w < REDUCE_WAVES; w++) total += part[w][threadIdx.x / 4][threadIdx.x % 4];
        if (col < gd) dgamma[col] = total;
        else dbeta[col - gd] = total;
    }
}

int grid_for(int64_t n_tokens, int tokens_per_block, int most) {
    const int64_t blocks = (n_tokens + tokens_per_block - 1) / tokens_per_block;
    return (int)(blocks < most ? blocks : most);
}

// Lets `Kernel` use what these kernels take of dynamic shared memory at most (with the backward's static arrays, the whole 160 KB would be more
// than there is, which the runtime refuses).  Asked for once per kernel; not a stream operation, so a graph that is being captured does not see it.
// The kernel is the parameter, not its type, which all instantiations share.
template <auto Kernel>
hipError_t allow_lds() {
    static hipError_t state = hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_FLOATS * (int)sizeof(float));
    return state;
}

template <typename T, int CPL, int LPT, bool GATED>
hipError_t launch_fwd_as(const Args& a, hipStream_t s) {
    const size_t lds = (size_t)2 * a.n_groups * a.row * sizeof(float);
    hipError_t e = allow_lds<fwd_kernel<T, CPL, LPT, GATED>>();
    if (e != hipSuccess) return e;
    const int grid = grid_for(a.n, WAVES * (CPL == 1 ? 2 : 1) * (64 / LPT), MAX_BLOCKS);
    hipLaunchKernelGGL((fwd_kernel<T, CPL, LPT, GATED>), dim3(grid), dim3(THREADS), lds, s, a);
    return hipGetLastError();
}

template <typename T, int CPL, int LPT, bool GATED, int NTHR>
hipError_t launch_bwd_form(const Args& a, int shares, hipStream_t s) {
    const size_t lds = (size_t)((GATED ? 2 : 1) + 2 * a.rep) * a.n_groups * a.row * sizeof(float);
    hipError_t e = allow_lds<bwd_kernel<T, CPL, LPT, GATED, NTHR>>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bwd_kernel<T, CPL, LPT, GATED, NTHR>), dim3(shares), dim3(NTHR), lds, s, a);
    return hipGetLastError();
}

template <typename T, int CPL, int LPT, bool GATED>
hipError_t launch_bwd_as(Args& a, int* shares, hipStream_t s) {
    constexpr int NT = 64 / LPT;
    const bool brief = is_brief(a.n, LPT);
    const int waves = (brief ? BRIEF_THREADS : bwd_threads(CPL)) / 64;
    // every wave of the grid gets one span when the tokens allow it, several passes of at most 64 and alike otherwise
    *shares = grid_for(a.n, waves * (brief ? 1 : NT), MAX_SHARES);
    const int64_t even = (a.n + (int64_t)*shares * waves - 1) / ((int64_t)*shares * waves), passes = (even + 63) / 64;
    a.span = (int32_t)((even + passes - 1) / passes);
    // accumulators for as many waves as end in the same group when groups are even, within 128 KB with the parameters
    const int room = (LDS_FLOATS / (a.n_groups * a.row) - (GATED ? 2 : 1)) / 2, want = (waves + a.n_groups - 1) / a.n_groups;
    a.rep = room < want ? room : want;
    if constexpr (NT > 1) {
        if (brief) return launch_bwd_form<T, CPL, LPT, GATED, BRIEF_THREADS>(a, *shares, s);
    }
    return launch_bwd_form<T, CPL, LPT, GATED, bwd_threads(CPL)>(a, *shares, s);
}

template <typename T, int CPL, int LPT, bool GATED>
hipError_t launch_as(int* shares, Args& a, hipStream_t s) {
    a.row = (a.d + LPT * 8 - 1) / (LPT * 8) * (LPT * 8);
    return shares ? launch_bwd_as<T, CPL, LPT, GATED>(a, shares, s) : launch_fwd_as<T, CPL, LPT, GATED>(a, s);
}

template <typename T, bool GATED>
hipError_t dispatch_width(int* shares, Args& a, hipStream_t s) {
    if (a.d <= 128) return launch_as<T, 1, 16, GATED>(shares, a, s);
    if (a.d <= 256) return launch_as<T, 1, 32, GATED>(shares, a, s);
    switch ((a.d + CHUNK - 1) / CHUNK) {
        case 1: return launch_as<T, 1, 64, GATED>(shares, a, s);
        case 2: return launch_as<T, 2, 64, GATED>(shares, a, s);
        case 3: return launch_as<T, 3, 64, GATED>(shares, a, s);
        default: return launch_as<T, 4, 64, GATED>(shares, a, s);
    }
}

// shares: null for the forward pass; for the backward pass, how many shares of dgamma / dbeta it leaves
hipError_t dispatch(int* shares, int dtype, Args& a, hipStream_t s) {
    const bool gated = a.gate != nullptr;
    if (dtype == MTFM_HTA_BF16) return gated ? dispatch_width<__bf16, true>(shares, a, s) : dispatch_width<__bf16, false>(shares, a, s);
    return gated ? dispatch_width<float, true>(shares, a, s) : dispatch_width<float, false>(shares, a, s);
}

int padded_row(int32_t d) { return (d + CHUNK - 1) / CHUNK * CHUNK; }

int check_shape(int64_t n_tokens, int32_t d, int32_t n_groups, int dtype) {
    if (dtype != MTFM_HTA_BF16 && dtype != MTFM_HTA_FP32)
        return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "dtype must be MTFM_HTA_BF16 or MTFM_HTA_FP32, got %d", dtype);
    if (n_tokens < 0) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "negative n_tokens");
    if (d <= 0 || d % 8 != 0)
        return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "d_model must be a positive multiple of 8, got %d", d);
    if (n_groups <= 0) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "n_groups must be positive, got %d", n_groups);
    if (d > CHUNK * MAX_CHUNKS)
        return hta::report_error(MTFM_HTA_ERR_UNSUPPORTED, "d_model %d exceeds %d", d, CHUNK * MAX_CHUNKS);
    if ((int64_t)n_groups * padded_row(d) > MAX_TABLE)
        return hta::report_error(MTFM_HTA_ERR_UNSUPPORTED,
                                 "n_groups (%d) x d_model rounded up to %d (%d) exceeds %d parameter slots in LDS", n_groups,
                                 CHUNK, padded_row(d), MAX_TABLE);
    return MTFM_HTA_OK;
}

bool misaligned(const void* p, unsigned a) { return ((uintptr_t)p & (a - 1)) != 0; }

}  // namespace gln

extern "C" {

int mtfm_gln_fwd(const void* x, const void* gate, const int32_t* group_id, const float* gamma, const float* beta,
                 void* y, float* mean, float* rstd, int64_t n_tokens, int32_t d_model, int32_t n_groups, float eps,
                 int dtype, void* stream) {
    if (int rc = gln::check_shape(n_tokens, d_model, n_groups, dtype)) return rc;
    if (!(eps >= 0.f)) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "eps must be >= 0");
    if (n_tokens == 0) return MTFM_HTA_OK;  // the arrays of an empty call may be null
    if (!x || !group_id || !gamma || !beta || !y) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "null pointer argument");
    if (gln::misaligned(x, 16) || gln::misaligned(gate, 16) || gln::misaligned(y, 16) || gln::misaligned(gamma, 16) ||
        gln::misaligned(beta, 16) || gln::misaligned(group_id, 4) || gln::misaligned(mean, 4) || gln::misaligned(rstd, 4))
        return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "x, gate, y, gamma, beta must be 16-byte aligned");
    gln::Args a = {};
    a.x = x, a.gate = gate, a.group_id = group_id, a.gamma = gamma, a.beta = beta, a.y = y, a.mean = mean, a.rstd = rstd;
    a.n = n_tokens, a.d = d_model, a.n_groups = n_groups, a.eps = eps;
    hipStream_t s = (hipStream_t)stream;
    hta::timing_begin(MTFM_GLN_KERNEL_FWD, s);
    const hipError_t e = gln::dispatch(nullptr, dtype, a, s);
    hta::timing_end(MTFM_GLN_KERNEL_FWD, s);
    if (e != hipSuccess) return hta::report_error(MTFM_HTA_ERR_LAUNCH, "gln forward launch: %s", hipGetErrorString(e));
    return MTFM_HTA_OK;
}

size_t mtfm_gln_bwd_workspace_bytes(int32_t d_model, int32_t n_groups) {
    if (gln::check_shape(0, d_model, n_groups, MTFM_HTA_BF16) != MTFM_HTA_OK) return 0;
    return (size_t)gln::WORKSPACE_SHARES * 2 * n_groups * d_model * sizeof(float);
}

int mtfm_gln_bwd(const void* dy, const void* x, const void* gate, const int32_t* group_id, const float* gamma,
                 const float* beta, const float* mean, const float* rstd, void* dx, void* dgate, float* dgamma,
                 float* dbeta, int64_t n_tokens, int32_t d_model, int32_t n_groups, int dtype, void* workspace,
                 size_t workspace_bytes, void* stream) {
    if (int rc = gln::check_shape(n_tokens, d_model, n_groups, dtype)) return rc;
    if (!dgamma || !dbeta) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "null pointer argument");
    // the per-token arrays of an empty call may be null
    if (n_tokens > 0 && (!dy || !x || !group_id || !gamma || !mean || !rstd || !dx))
        return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "null pointer argument");
    if ((gate == nullptr) != (dgate == nullptr))
        return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "gate and dgate must both be given or both be NULL");
    if (gate && !beta) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "beta is required with a gate");
    if (gln::misaligned(dy, 16) || gln::misaligned(x, 16) || gln::misaligned(gate, 16) || gln::misaligned(dx, 16) ||
        gln::misaligned(dgate, 16) || gln::misaligned(gamma, 16) || gln::misaligned(beta, 16) ||
        gln::misaligned(dgamma, 4) || gln::misaligned(dbeta, 4) || gln::misaligned(mean, 4) || gln::misaligned(rstd, 4) ||
        gln::misaligned(group_id, 4))
        return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "dy, x, gate, dx, dgate, gamma, beta must be 16-byte aligned");
    const size_t need = mtfm_gln_bwd_workspace_bytes(d_model, n_groups);
    if (!workspace || workspace_bytes < need)
        return hta::report_error(MTFM_HTA_ERR_WORKSPACE, "this call needs %zu bytes of workspace, got %zu", need,
                                 workspace ? workspace_bytes : (size_t)0);
    if (gln::misaligned(workspace, 256)) return hta::report_error(MTFM_HTA_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    gln::Args a = {};
    a.dy = dy, a.x = x, a.gate = gate, a.group_id = group_id, a.gamma = gamma, a.beta = beta, a.mean_in = mean, a.rstd_in = rstd;
    a.dx = dx, a.dgate = dgate, a.partials = (float*)workspace;
    a.n = n_tokens, a.d = d_model, a.n_groups = n_groups;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipSuccess;
    int shares = 0;
    if (n_tokens > 0) {
        hta::timing_begin(MTFM_GLN_KERNEL_BWD, s);
        e = gln::dispatch(&shares, dtype, a, s);
        hta::timing_end(MTFM_GLN_KERNEL_BWD, s);
        if (e != hipSuccess) return hta::report_error(MTFM_HTA_ERR_LAUNCH, "gln backward launch: %s", hipGetErrorString(e));
    }
    const int gd = n_groups * d_model;
    hta::timing_begin(MTFM_GLN_KERNEL_BWD_REDUCE, s);
    hipLaunchKernelGGL(gln::reduce_kernel, dim3((2 * gd + gln::REDUCE_COLS - 1) / gln::REDUCE_COLS),
                       dim3(gln::REDUCE_THREADS), 0, s, (const float*)workspace, shares, gd, dgamma, dbeta);
    e = hipGetLastError();
    hta::timing_end(MTFM_GLN_KERNEL_BWD_REDUCE, s);
    if (e != hipSuccess) return hta::report_error(MTFM_HTA_ERR_LAUNCH, "gln reduce launch: %s", hipGetErrorString(e));
    return MTFM_HTA_OK;
}

int mtfm_gln_validate_host(const int32_t* group_id, int64_t n_tokens, int32_t n_groups) {
    if (n_tokens < 0 || n_groups <= 0) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "negative n_tokens or n_groups <= 0");
    if (n_tokens > 0 && !group_id) return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "null array");
    for (int64_t i = 0; i < n_tokens; i++)
        if (group_id[i] < 0 || group_id[i] >= n_groups)
            return hta::report_error(MTFM_HTA_ERR_INVALID_ARG, "token %lld: group id %d outside [0, %d)", (long long)i,
                                     group_id[i], n_groups);
    return MTFM_HTA_OK;
}

}  // extern "C"
