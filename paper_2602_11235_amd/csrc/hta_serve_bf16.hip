// bf16 forward pass of Hybrid Target Attention for a handful of requests (gfx950): one user's history and the
// candidates of a scenario, or a few of them in one call.  Same mask and products as hta_fwd_bf16.hip; what differs is
// what bounds it: the work of a call is a few microseconds of the chip, so latencies count and not rates.
//
// Work decomposition: one workgroup = (user, kv head, RW * RB blocks of 32 packed (row, head) pairs, key split).  Its eight
// waves are RW row groups x KW key ways: the waves of a row group take every KW-th block of keys, each with a softmax
// of its own, and merge their results through LDS at the end.  Splitting the keys inside the workgroup costs no memory
// traffic and no second launch, so it comes first; only when that leaves units idle long enough to pay for the merge
// launch are the keys split over workgroups as well.
// With RW = 1 no two waves read the same key: nothing is shared, a wave waits for its own copies only and the key loop
// has no barrier.  K and V travel global -> LDS asynchronously; the K of the next block is requested when the scores of
// this one have been formed, its V when the products have.
//
// What bounds it, at head_dim 64 and one workgroup of 32 rows per compute unit: 2.05 us per 1000 keys, where the copies
// alone take 1.66 (64 bytes per clock and unit) and the arithmetic alone 2.0, and 6 us of launch, first loads and merge.  K
// fragments straight to registers (no LDS write and read): 3.6 us per 1000 keys, 32-byte pieces of a row per lane pair.
// Four waves with the whole register file each: 5 to 6 us.  One 2048 + 128 token request at 8/2 heads: 18.0 -> 10.2 us
// per call; 8 requests of 512..4096: 22.1 -> 16.3, with real-time tokens 25.0 -> 16.3; 4 of 8192 at head_dim 128: 37.6 -> 32.8.
#include "../../include/mtfm_hta.h"
#include "../../include/mtfm_hta_timing.h"
#include "hta_common.h"
#include "hta_fwd_rows.h"
#include "hta_mfma.h"
#include "hta_tiles.h"

#include <algorithm>
#include <cmath>

namespace hta {
namespace {

constexpr int SUB = 32;  // keys of a sub-tile

// SPS: 32-key sub-tiles per step (two of them interleave what each waits for); NST: steps resident in LDS.  K and V of a
// step are requested as soon as their predecessors in the slot have been read, which with NST = 1 is half a step ahead.
template <int D, int RB, int RW, int NW, int SPS, int NST>
struct Serve {
    static constexpr int BLK = SUB * SPS;              // keys of a step
    static constexpr int TILE = BLK * D;               // elements of its K or V
    static constexpr int CPR = D / 8;                  // 16-byte chunks per row
    static constexpr int RPC = 64 / CPR;               // rows per 1 KB copy
    static constexpr int KW = NW / RW;                 // key ways
    static constexpr int COPIES = BLK / RPC / RW;      // copies per wave of its K, and of its V
    static constexpr int ROWS = RW * RB * SUB;         // packed rows of the workgroup
    static constexpr int Q_COPIES = ROWS / RPC;        // copies of their Q, dealt to the waves
    static constexpr int QUADS = D / 4, MERGED = RW * SUB * QUADS;  // 4 features each, of a row block
    static constexpr int NIT = (MERGED + NW * 64 - 1) / (NW * 64);               // a thread's share of them
    static constexpr int PITCH = D + 4;                // floats per row of the merge buffer (16-byte words spread over the banks)
    static constexpr int MERGE_BYTES = NW * SUB * (PITCH + 2) * 4;
    static constexpr int KV_BYTES = KW * NST * 2 * TILE * 2;
    static constexpr int Q = KV_BYTES, BEFORE = Q + ROWS * D * 2;
    static constexpr int BYTES = BEFORE > MERGE_BYTES ? BEFORE : MERGE_BYTES;
};
constexpr int TS_CAP = 512;  // real-time tokens of a user whose timestamps are searched in LDS

// How a launch's workgroups map to work, with what takes the place of divisions in the kernel (a workgroup of a small call lives for 3 us,
// of which the divisions of a general decode took 0.3).  Grid: x = XCD + 8 * (tile / spread), y = group / 8.  A group is (user, kv
// head, head chunk, split, one of `spread` shares of the tiles): its row tiles read the same keys and stay on one XCD, the splits of an item
// go to different ones.
struct ServeGrid {
    uint32_t n_groups, spread_log2;       // spread: 1 or 2
    uint32_t ny, ny_magic;               // groups of a user; 2^32 / ny, rounded up (0: ny is 1)
    uint32_t n_splits, splits_magic;     // likewise
    int32_t per;                         // blocks of keys per split
};
inline uint32_t div_magic(uint32_t d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / d + 1); }
// n / d for n d < 2^32
__device__ inline uint32_t div_by(uint32_t n, uint32_t magic) { return magic == 0 ? n : __umulhi(n, magic); }

// The arrays that the first loads go to and what finds the user stand alone at the front: arguments in scalar registers when the kernel
// starts (build.py, KERNARG_PRELOAD), while those inside Params take a load that costs 0.45 us at the start of a launch.
template <int D, int RB, int RW, int NW, int SPS, int NST, bool RT, bool PW>
__global__ __launch_bounds__(NW * 64, NW / 4) void serve_kernel(const int32_t* hist_len, const int32_t* n_targets, const int32_t* q_off,
                                                                const int32_t* kv_off, const int32_t* rt_len, uint32_t ny, uint32_t ny_magic,
                                                                ServeGrid sg, Params p, RowMap map) {
    using SV = Serve<D, RB, RW, NW, SPS, NST>;
    constexpr int BLK = SV::BLK, CP = SV::COPIES, KW = SV::KW, QUADS = SV::QUADS, NIT = SV::NIT;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SV::BYTES];
    __shared__ __attribute__((aligned(256))) int ts_s[RT ? TS_CAP : 1], row_ts[RT ? SV::ROWS * 2 : 1];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const uint32_t group = blockIdx.y * N_XCD + blockIdx.x % N_XCD;
    if (group >= sg.n_groups) return;
    const int b = (int)div_by(group, ny_magic);
    const int L = hist_len[b], T = n_targets[b], R = RT ? rt_len[b] : 0;
    const int64_t q_base = q_off[b], kv_base = kv_off[b];
    const uint32_t y = (group - (uint32_t)b * ny) >> sg.spread_log2;
    const int tile = (int)((blockIdx.x / N_XCD << sg.spread_log2) + (group & ((1u << sg.spread_log2) - 1u)));
    const int gc = (int)div_by(y, sg.splits_magic), split = (int)y - gc * (int)sg.n_splits;
    const int g = map.n_chunks == 1 ? gc : gc / map.n_chunks, chunk = gc - g * map.n_chunks;
    const int LK = L + R;  // keys that run through the tile loop: history, then real-time
    const int n_rows = p.layer == 0 ? LK + T : T;
    const int n_all = (LK + BLK - 1) / BLK, lo = min(split * sg.per, n_all), hi = min(lo + sg.per, n_all);
    if (tile * map.rows >= n_rows) return;  // uniform for the whole workgroup
    const PackedRows pr(map, tile, chunk, n_rows, g, p.Hq / p.Hkv);
    if (!PW && split > 0 && lo >= n_all) {  // a user whose keys end before this split
        const PackedRows::Row x = pr.at(tid);
        if (tid < SV::ROWS && x.live) p.lse_part[((int64_t)split * p.Hq + x.h) * p.total_q + q_base + x.row] = -INFINITY;
        return;
    }
    const int tok_shift = p.layer == 0 ? 0 : LK;  // token index of query row 0
    const int rw = wave / KW, kw = wave % KW, rho0 = rw * RB * 32;
    const bool wave_live = RW == 1 || pr.any_from(rho0);
    const int n_mine = hi - lo > kw ? (hi - lo - kw + KW - 1) / KW : 0;  // steps of this key way: blocks lo + kw + i KW

    // K or V of step i to its slot.  Keys past the end repeat the last one (their weight is forced to zero).
    const __bf16* kg = (const __bf16*)p.k + (int64_t)g * D;
    const __bf16* vg = (const __bf16*)p.v + (int64_t)g * D;
    uint32_t voff[CP];  // byte offsets of the chunks this lane fetches from the first element of the block
#pragma unroll
    for (int j = 0; j < CP; j++) {
        const int trow = (j * RW + rw) * SV::RPC + lane / SV::CPR;
        voff[j] = (uint32_t)((trow * p.Hkv * D + ((lane % SV::CPR) ^ swizzle<D>(trow)) * 8) * 2);
    }
    auto slot = [&](int i) __attribute__((always_inline)) { return (kw * NST + (NST == 1 ? 0 : i % NST)) * (2 * SV::TILE * 2); };
    auto fetch = [&](const __bf16* src, int i, int part) __attribute__((always_inline)) {
        if (i >= n_mine) return;
        const int k0 = (lo + kw + i * KW) * BLK;
        const __bf16* base = src + (kv_base + k0) * p.Hkv * D;
        const uint32_t dst = lds_address(smem) + (uint32_t)(slot(i) + part * SV::TILE * 2);
        if (k0 + BLK <= LK) {
#pragma unroll
            for (int j = 0; j < CP; j++) copy16_global_to_lds_at(base, voff[j], dst + (j * RW + rw) * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < CP; j++) {
                const int trow = (j * RW + rw) * SV::RPC + lane / SV::CPR;
                const uint32_t past = (uint32_t)max(trow - (LK - 1 - k0), 0);
                copy16_global_to_lds_at(base, voff[j] - past * (uint32_t)(p.Hkv * D * 2), dst + (j * RW + rw) * 1024);
            }
        }
    };
    // (from the tile's first row on 32 bits suffice for a lane's offset)
    const __bf16* const q_tile = (const __bf16*)p.q + (q_base + pr.row0) * p.Hq * D;
    const int64_t own_tile = ((kv_base + tok_shift + pr.row0) * p.Hkv + g) * D;
    // What the rows need comes first, the K and V behind it: 128 KB of copies per unit take their time to be issued alone.
    if constexpr (RT) {
        if (R <= TS_CAP && wave * 64 < R && wave < TS_CAP / 64)
            copy4_global_to_lds_at(p.ts + kv_base + L + min(wave * 64 + lane, R - 1), lds_address(ts_s) + wave * 256u);
        if (wave < SV::ROWS / 32)  // (one row to two lanes)
            copy4_global_to_lds_at(p.ts + kv_base + tok_shift + pr.at(wave * 32 + l32).row, lds_address(row_ts) + wave * 256u);
    }
    for (int j = wave; j < SV::Q_COPIES; j += NW) {
        const int trow = j * SV::RPC + lane / SV::CPR;
        const PackedRows::Row x = pr.at(trow);
        copy16_global_to_lds_at(q_tile, (uint32_t)(((x.row - pr.row0) * p.Hq + x.h) * D + ((lane % SV::CPR) ^ swizzle<D>(trow)) * 8) * 2u,
                                lds_address(smem) + (uint32_t)(SV::Q + j * 1024));
    }
    // The own key of target rows (rule 3) and of real-time rows joins in the merge: its logit and weight are formed by the threads that
    // hold 4 features of the row there.  Requested here, used behind the key loop.
    bf16x4 own_q[RB][NIT], own_k[RB][NIT], own_v[RB][NIT];
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            own_q[rb][it] = own_k[rb][it] = own_v[rb][it] = bf16x4{};
            if (split == 0) {
                const int id = tid + it * NW * 64, c = id % QUADS, rl = id / QUADS;
                const PackedRows::Row x = pr.at((rl / SUB * RB + rb) * 32 + rl % SUB);
                const uint32_t koff = (uint32_t)((x.row - pr.row0) * p.Hkv * D + 4 * c);
                own_q[rb][it] = *(const bf16x4*)(q_tile + (uint32_t)(((x.row - pr.row0) * p.Hq + x.h) * D + 4 * c));
                own_k[rb][it] = *(const bf16x4*)((const __bf16*)p.k + own_tile + koff);
                own_v[rb][it] = *(const bf16x4*)((const __bf16*)p.v + own_tile + koff);
            }
        }
#pragma unroll
    for (int i = 0; i < NST; i++) {
        fetch(kg, i, 0);
        fetch(vg, i, 1);
    }

    FwdRows<D, RB, RT, PW> rows;
    rows.init_lane(p, lane);
    rows.reset();
    if (n_mine >= NST) wait_vmem_outstanding<2 * CP * NST>(); else wait_vmem_outstanding<0>();
    lds_barrier();
    rows.take_q((const __bf16*)(smem + SV::Q) + rw * RB * SUB * D, L);
    if constexpr (RT) {
        // mask rule 2: the row sees the history and the real-time tokens strictly earlier than itself, a prefix
        const int32_t* ts = p.ts + kv_base + L;
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const int t = row_ts[(rw * RB + rb) * 64 + lane];
            int a = 0, e = R;
            while (a < e) {
                const int mid = (a + e) >> 1;
                const int v = R <= TS_CAP ? ts_s[mid] : ts[mid];
                if (v < t) a = mid + 1; else e = mid;
            }
            rows.lim[rb] = L + a;
        }
    }

    // wait until at most n steps' K and V, and then (Half: V, or the K of one more step), are in flight
    auto wait_copies = [&](int steps, bool half) __attribute__((always_inline)) {
        if (NST > 1 && steps >= 1) {
            if (half) wait_vmem_outstanding<3 * CP>(); else wait_vmem_outstanding<2 * CP>();
        } else {
            if (half) wait_vmem_outstanding<CP>(); else wait_vmem_outstanding<0>();
        }
    };
    static_assert(NST <= 2, "wait_copies");
    auto step = [&](int i, auto Tail) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(Tail)::value;
        const int k0 = (lo + kw + i * KW) * BLK, left = n_mine - 1 - i;
        const __bf16* Ks = (const __bf16*)(smem + slot(i));
        floatx16 S[SPS][RB];
        const bool work = wave_live && (RW == 1 || i < n_mine);
        wait_copies(min(NST - 1, left), true);  // newer than K_i: V_i and the following steps
        if (RW > 1) lds_barrier();
        if (work) rows.template scores<SPS>(S, Ks);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // K_i has been read
        if (RW > 1) {
            wait_copies(min(NST - 1, left), false);
            lds_barrier();
        }
        fetch(kg, i + NST, 0);
        if (RW == 1) wait_copies(min(NST - 1, left), left >= NST);  // newer than V_i: the following steps, and K_(i + NST)
        if (work) rows.template absorb<TAIL, SPS>(S, Ks + SV::TILE, LK - k0, k0, L);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (RW > 1) lds_barrier();
        fetch(vg, i + NST, 1);
    };
    // blocks of history keys first, then those that need a mask (the last one; more with real-time tokens)
    const int n_rounds = RW == 1 ? n_mine : (hi - lo + KW - 1) / KW;  // (barriers: the same number of steps for every wave)
    const int n_whole = RW == 1 ? min(max(min(hi, L / BLK) - lo - kw + KW - 1, 0) / KW, n_mine) : max(min(hi, L / BLK) - lo, 0) / KW;
    for (int i = 0; i < n_whole; i++) step(i, std::false_type{});
    for (int i = n_whole; i < n_rounds; i++) step(i, std::true_type{});

    // ---- the own keys' logits, summed over the threads of a row: log2 units (PW: the weight itself), -inf (0) where there is none
    float own[RB][NIT];
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int rl = (tid + it * NW * 64) / QUADS;
            const bool has = split == 0 && tok_shift + pr.at((rl / SUB * RB + rb) * 32 + rl % SUB).row >= L;
            float dot = dot_bf16x4(0.f, own_q[rb][it], own_k[rb][it]);
            dot = sum_lanes<QUADS>(dot);
            own[rb][it] = PW ? (has ? pw_silu(dot, pw_sigmoid(dot, rows.neg_c2)) : 0.f) : (has ? dot * rows.c2 : -INFINITY);
        }
    // ---- merge the waves' results through LDS, one row block after the other
    float* acc = (float*)smem;                          // [wave][row][PITCH]
    float* stat = acc + NW * SUB * SV::PITCH;           // [wave][row][m, l]
    static_for<0, RB>([&](auto Rb) {
    constexpr int rb = decltype(Rb)::value;
    lds_barrier();  // every wave has read its last block (or the previous row block)
    {
        const float lt = rows.l[rb] + other_half(rows.l[rb]);
        if (hf == 0) {
            stat[(wave * SUB + l32) * 2] = rows.m[rb];
            stat[(wave * SUB + l32) * 2 + 1] = lt;
        }
        float* o = acc + (wave * SUB + l32) * SV::PITCH + 4 * hf;
#pragma unroll
        for (int db = 0; db < D / 32; db++)
#pragma unroll
            for (int v4 = 0; v4 < 4; v4++) {
                floatx4 x;
#pragma unroll
                for (int j = 0; j < 4; j++) x[j] = rows.O[rb][db][4 * v4 + j];
                *(floatx4*)(o + db * 32 + 8 * v4) = x;
            }
    }
    lds_barrier();
#pragma unroll
    for (int it = 0; it < NIT; it++) {
        const int id = tid + it * NW * 64;
        const int c = id % QUADS, rl = id / QUADS, l = rl % SUB, w0 = rl / SUB % RW * KW;  // 4 features of a row; its first wave
        const PackedRows::Row x = pr.at((rl / SUB * RB + rb) * 32 + l);
        float mx = PW ? 0.f : fmaxf(own[rb][it], -1e30f);
        float2 ml[KW];
        if constexpr (!PW) {
#pragma unroll
            for (int k = 0; k < KW; k++) {
                ml[k] = *(const float2*)(stat + ((w0 + k) * SUB + l) * 2);
                mx = fmaxf(mx, ml[k].x);
            }
        }
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
        float sum = 0.f;
        if (PW || own[rb][it] > -INFINITY) {
            const float f = PW ? own[rb][it] : fast_exp2(own[rb][it] - mx);
            sum = f;
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = f * (float)own_v[rb][it][j];
        }
#pragma unroll
        for (int k = 0; k < KW; k++) {
            const float f = PW ? 1.f : fast_exp2(ml[k].x - mx);  // 0 for a wave that saw no key
            const floatx4 ok = *(const floatx4*)(acc + ((w0 + k) * SUB + l) * SV::PITCH + 4 * c);
            if constexpr (!PW) sum = fmaf(f, ml[k].y, sum);
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = fmaf(f, ok[j], o[j]);
        }
        if (!x.live || id >= SV::MERGED) continue;
        const float inv = PW ? p.norm * p.scale : (sum > 0.f ? 1.f / sum : 0.f);
        const float lse = sum > 0.f ? (mx + __builtin_amdgcn_logf(sum)) * LN2 : -INFINITY;
        const int64_t row = q_base + x.row;
        if (sg.n_splits == 1) {
            bf16x4 o4;
#pragma unroll
            for (int j = 0; j < 4; j++) o4[j] = (__bf16)(o[j] * inv);
            *(bf16x4*)((__bf16*)p.out + (row * p.Hq + x.h) * D + 4 * c) = o4;
            if (!PW && c == 0) p.lse[(int64_t)x.h * p.total_q + row] = lse;
        } else {
            floatx4 o4;
#pragma unroll
            for (int j = 0; j < 4; j++) o4[j] = o[j] * inv;
            *(floatx4*)(p.o_part + (((int64_t)split * p.total_q + row) * p.Hq + x.h) * D + 4 * c) = o4;
            if (!PW && c == 0) p.lse_part[((int64_t)split * p.Hq + x.h) * p.total_q + row] = lse;
        }
    }
    });
}

// out = sum_s w_s O_s / sum_s w_s with w_s = exp(lse_s - max lse), lse = max lse + log sum_s w_s: the exact
// combination of softmax results over disjoint key sets.  One thread per 4 features of a (row, head).
// PW: the partial results are partial sums of non-normalised weights: out = sum_s O_s, no lse.
// All loads of a thread travel together, AT_ONCE splits of them: one trip to memory is most of what this launch takes.  (Split after split,
// as the remainder of an unrolled loop is: 2 us more for 4 splits.)
template <int D, int AT_ONCE, bool PW>
__global__ __launch_bounds__(256) void merge_splits_kernel(const float* o_part, const float* lse_part, int64_t total_q, int Hq, int n_splits,
                                                           void* out, float* lse) {
    constexpr int QUADS = D / 4;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= total_q * Hq * QUADS) return;
    const uint32_t rh = (uint32_t)(id / QUADS), row = rh / (uint32_t)Hq, h = rh - row * (uint32_t)Hq;  // (both below 2^31)
    const int64_t at_lse = (int64_t)h * total_q + row, l_stride = (int64_t)Hq * total_q, o_stride = total_q * Hq * D;
    floatx4 o = {0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, sum = 0.f;
    for (int s0 = 0; s0 < n_splits; s0 += AT_ONCE) {
        floatx4 os[AT_ONCE];
        float ls[AT_ONCE];
#pragma unroll
        for (int s = 0; s < AT_ONCE; s++) {  // (behind the last one: the last one again)
            const int i = min(s0 + s, n_splits - 1);
            ls[s] = PW ? 0.f : lse_part[at_lse + i * l_stride];
            os[s] = *(const floatx4*)(o_part + id * 4 + i * o_stride);
        }
        const float before = mx;
        if constexpr (!PW) {
#pragma unroll
            for (int s = 0; s < AT_ONCE; s++) mx = fmaxf(mx, ls[s]);
            const float f = before > -INFINITY ? __expf(before - mx) : 0.f;
            sum *= f;
            o *= f;
        }
#pragma unroll
        for (int s = 0; s < AT_ONCE; s++) {
            const float w = s0 + s >= n_splits ? 0.f : PW ? 1.f : __expf(ls[s] - mx);
            sum += w;
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = s0 + s >= n_splits || (!PW && ls[s] == -INFINITY) ? o[j] : fmaf(w, os[s][j], o[j]);  // (-inf: nothing was left)
        }
    }
    const float inv = PW ? 1.f : 1.f / sum;
    bf16x4 o4;
#pragma unroll
    for (int j = 0; j < 4; j++) o4[j] = (__bf16)(o[j] * inv);
    *(bf16x4*)((__bf16*)out + id * 4) = o4;
    if (!PW && id % QUADS == 0) lse[at_lse] = mx + __logf(sum);
}

template <int D, int RB, int RW, int NW, int SPS, int NST>
hipError_t launch(const Params& p, hipStream_t s) {
    auto kernel = serve_kernel<D, RB, RW, NW, SPS, NST, false, false>;
    if (p.pointwise)
        kernel = p.rt_len ? serve_kernel<D, RB, RW, NW, SPS, NST, true, true> : serve_kernel<D, RB, RW, NW, SPS, NST, false, true>;
    else if (p.rt_len)
        kernel = serve_kernel<D, RB, RW, NW, SPS, NST, true, false>;
    const int64_t rows = max_query_rows(p);
    if (rows <= 0) return hipSuccess;
    const RowMap map = row_map(RW * RB * 32, p.Hq, p.Hkv, rows);
    const int64_t max_blocks = (max_lead_keys(p) + SUB * SPS - 1) / (SUB * SPS);
    ServeGrid sg;
    sg.per = (int32_t)std::max<int64_t>((max_blocks + p.n_splits - 1) / p.n_splits, 1);
    sg.n_splits = (uint32_t)std::max<int64_t>((max_blocks + sg.per - 1) / sg.per, 1);
    // One XCD per group is best for its L2; two when there are so few groups that an XCD of 32 units can get more
    // workgroups than it has units while others idle (14 requests of 1053 keys, 28 groups: 23 -> 14 us).
    const int64_t groups = (int64_t)p.batch * p.Hkv * map.n_chunks * sg.n_splits;
    const int spread = groups < 64 && (groups + N_XCD - 1) / N_XCD * map.n_tiles > 32 ? 2 : 1;
    sg.ny = (uint32_t)(groups / p.batch * spread);
    sg.spread_log2 = spread / 2;
    sg.n_groups = sg.ny * (uint32_t)p.batch;
    sg.ny_magic = div_magic(sg.ny);
    sg.splits_magic = div_magic(sg.n_splits);
    const int64_t nx = (int64_t)((map.n_tiles + spread - 1) / spread) * N_XCD, n_y = (sg.n_groups + N_XCD - 1) / N_XCD;
    if (nx * n_y >= (1ll << 31) || n_y > 65535 || (int64_t)sg.n_groups * sg.ny >= (1ll << 32)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel, dim3((unsigned)nx, (unsigned)n_y), dim3(NW * 64), 0, s, p.hist_len, p.n_targets, p.q_off, p.kv_off, p.rt_len, sg.ny,
                       sg.ny_magic, sg, p, map);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || sg.n_splits == 1) return e;
    const int64_t threads = p.total_q * p.Hq * (p.d / 4);
    auto merge = merge_splits_kernel<D, 8, false>;
    if (p.pointwise) merge = sg.n_splits <= 2 ? merge_splits_kernel<D, 2, true> : sg.n_splits <= 4 ? merge_splits_kernel<D, 4, true> : merge_splits_kernel<D, 8, true>;
    else if (sg.n_splits <= 4) merge = sg.n_splits <= 2 ? merge_splits_kernel<D, 2, false> : merge_splits_kernel<D, 4, false>;
    hipLaunchKernelGGL(merge, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       p.o_part, p.lse_part, p.total_q, p.Hq, (int)sg.n_splits, p.out, p.lse);
    return hipGetLastError();
}

// workgroups with work to do: `lanes` packed rows each, from the bounds and the number of query rows of the call
int64_t live_tiles(const Params& p, int lanes) {
    const RowMap map = row_map(lanes, p.Hq, p.Hkv, max_query_rows(p));
    const int64_t groups = (int64_t)p.batch * p.Hkv * map.n_chunks;
    return std::min(groups * map.n_tiles, p.total_q * p.Hkv * map.n_chunks / map.rows + groups / 2);
}

// The shape of a call's workgroups.  Blocks of 32 rows finish soonest while every one gets a unit to itself; once they
// queue up, 64 rows per workgroup (two row blocks per wave at head_dim 64, two row groups sharing their keys at 128, where
// the registers do not hold two) halve the traffic of the copies.
enum Shape { ROWS32, ROWS64 };
Shape shape_of(const Params& p) { return p.d > 32 && live_tiles(p, 32) > (p.d == 64 ? 256 : 512) ? ROWS64 : ROWS32; }

}  // namespace

// What the workspace formula below counts, which is part of the interface's contract: tiles of 128, 256 or 512 rows, fewer heads per
// tile where a group does not divide evenly.  (Not what any kernel launches today: see fwd_workgroup_rows for that.)
static int64_t ordinary_items(int32_t batch, int32_t Hq, int32_t Hkv, int32_t d, int64_t max_rows) {
    const int64_t r = Hq / Hkv, waves = r % 4 == 0 ? 8 : 4;
    const int64_t lanes = 32 * waves * (d == 32 || (d == 64 && waves == 4) ? 2 : 1);
    const int64_t heads = r % waves == 0 ? waves : (r % 4 == 0 ? 4 : (r % 2 == 0 ? 2 : 1));
    return batch * Hkv * (r / heads) * ((max_rows + lanes / heads - 1) / (lanes / heads));
}

// The workspace of a forward call has room for this many partial results per row.
int fwd_key_splits(int32_t batch, int32_t Hq, int32_t Hkv, int32_t d, int64_t max_rows, int64_t max_keys) {
    constexpr int64_t CUS = 256, MIN_TILES = 4, MAX_SPLITS = 32;
    if (batch <= 0 || max_rows <= 0 || !bf16_supported(d, Hq, Hkv)) return 1;
    const int64_t items = ordinary_items(batch, Hq, Hkv, d, max_rows);
    if (items >= CUS) return 1;
    const int64_t want = (CUS + items - 1) / items, by_len = ((max_keys + 63) / 64) / MIN_TILES;
    int64_t n = want < by_len ? want : by_len;
    n = n < MAX_SPLITS ? n : MAX_SPLITS;
    return n > 1 ? (int)n : 1;
}

// Estimated times of a call (us) with the keys in one piece, from fits of 2700 calls on both sides of the line (1 to 400 users,
// 4 to 256 candidates or a full layer, 64 to 8192 keys, all of one length or spread over a factor of 8; with and without
// real-time tokens and with pointwise weights).  The ordinary kernel, up to a workgroup per unit: the longest one, a little more the
// fuller the chip, and the schedule and limits launches as they were then: 0.02 us per user, which 32 users hardly see, and 2 us with real-time
// tokens, whose launch is gone.  (That leaves the ordinary kernel out of some calls where it is the faster one.  Without the 2 us 860 of
// 3999 calls with real-time tokens near the line change sides: 0.87 of the time on average, but 228 of them slower, by half at
// most; the kernel for a few requests takes 3 us longer with real-time tokens than estimated.  Both want a fit of their own.)
static double ordinary_us(const Params& p, int64_t workgroups) {
    struct { double launch, key, key_full; } c;
    if (p.d == 32) c = {6.2, 9.5e-3, 3.5e-3};
    else if (p.d == 128) c = {9.6, 17.6e-3, 4.e-3};
    else if (fwd_workgroup_rows(p) == 128) c = {7.5, 13.e-3, 2.5e-3};
    else c = {8., 14.e-3, 5.e-3};
    return c.launch + 0.02 * p.batch + (p.rt_len ? 2. : 0.) + c.key * max_lead_keys(p) + c.key_full * mean_keys(p) * workgroups / 256.;
}
// The kernel above: one workgroup per unit, so rounds of 256 of them.
static double serve_us(const Params& p, Shape shape) {
    struct { double launch, fixed, key; } c;
    if (p.d == 32) c = {1., 3.7, 2.7e-3};
    else if (p.d == 64 && shape == ROWS64) c = {1., 7., 5.2e-3};
    else if (p.d == 64) c = {3., 2.5, 3.e-3};
    else if (shape == ROWS64) c = {1., 9., 10.e-3};
    else c = {0., 7., 5.3e-3};
    const double longest = (double)max_lead_keys(p), mean = mean_keys(p), full = live_tiles(p, shape == ROWS64 ? 64 : 32) / 256.;
    const double rounds = mean > 0.9 * longest ? std::ceil(full) : std::max(1., full + 0.75);
    return c.launch + c.fixed * rounds + c.key * std::max(longest, mean * rounds);
}

// This kernel or the ordinary one, which shares each K/V tile among 128 or 256 rows and keeps two workgroups on a unit.  Once its
// workgroups nearly fill the chip, the ordinary one (at head_dim 64, 224 to 330 of them: on average 1.2 times as fast, though
// not on long histories of unlike lengths; 128: 1.3; 32, 448 to 600: 1.5).  Below that, keys are split over workgroups when the time
// this takes off the longest item is worth the merge: per key and workgroup 2.05 ns at head_dim 64, 4.4 at 128; merge 4.2 us,
// partial results at 3 TB/s.  Where it is not, by the estimates above: 64-row workgroups that come in rounds lose to 256-row ones
// that do not.  (8/2 heads of 64: 27 users x 256 candidates on 512 keys 38 us here against 20 there, on 2048 64 / 45; 13 users on
// 2048 34 / 43; 40 users x 128 candidates, 16/2 heads of 128, 64..512 keys 60 / 31; 110 x 256, 4/2 heads of 32, 512 keys 63 / 25.
// Of the 2700 calls 622 had a tenth or more to gain on the other side when only full chips went there, 47 have now.)
int serve_splits(const Params& p, int room) {
    const int64_t ordinary = live_tiles(p, fwd_workgroup_rows(p));
    if (ordinary >= (p.d == 32 ? 448 : 224)) return 0;
    const Shape shape = shape_of(p);
    if (room > 1 && shape != ROWS64) {
        const RowMap map = row_map(32, p.Hq, p.Hkv, max_query_rows(p));
        const int64_t items = (int64_t)p.batch * p.Hkv * map.n_chunks * map.n_tiles;
        const double loop = max_lead_keys(p) * (p.d == 128 ? 4.4e-3 : 2.05e-3);
        const double part = 2.0 * p.total_q * p.Hq * p.d * 4 / 3e6;
        int best = 1;
        double best_us = loop;
        for (int s = 2; s <= room && items * s <= 256; s++) {
            const double us = loop / s + 4.2 + s * (part + 0.05);
            if (us < best_us) best = s, best_us = us;
        }
        if (best > 1) return best;
    }
    return ordinary_us(p, ordinary) < 0.97 * serve_us(p, shape) ? 0 : 1;
}

hipError_t launch_serve_bf16(const Params& p, hipStream_t s) {
    const Shape shape = shape_of(p);
    // short lists of keys per wave: single sub-tiles divide more evenly than pairs
    const bool brief = max_lead_keys(p) / p.n_splits <= 1024;
    hipError_t e;
    timing_begin(MTFM_HTA_KERNEL_FWD, s);
    switch (p.d) {
        case 32: e = launch<32, 1, 1, 8, 2, 2>(p, s); break;
        case 64: e = shape == ROWS64 ? launch<64, 2, 1, 8, 1, 2>(p, s) : brief ? launch<64, 1, 1, 8, 1, 2>(p, s) : launch<64, 1, 1, 8, 2, 1>(p, s); break;
        case 128: e = shape == ROWS64 ? launch<128, 1, 2, 8, 2, 1>(p, s) : launch<128, 1, 1, 8, 1, 1>(p, s); break;
        default: e = hipErrorInvalidValue;
    }
    timing_end(MTFM_HTA_KERNEL_FWD, s);
    return e;
}

}  // namespace hta
