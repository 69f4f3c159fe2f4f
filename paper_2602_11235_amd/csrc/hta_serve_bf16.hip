// bf16 forward pass of Hybrid Target Attention for a handful of requests (gfx950): one user's history and the
// candidates of a scenario, or a few of them in one call.  Same mask and products as hta_fwd_bf16.hip; what differs is
// what bounds it: the work of a call is a few microseconds of the chip, so latencies count and not rates.
//
// Work decomposition: one workgroup = (user, kv head, one or two blocks of 32 packed (row, head) pairs, key split).  Its eight waves
// take every eighth block of keys, each with a softmax of its own, and merge their results through LDS at the end.  Splitting the
// keys inside the workgroup costs no memory traffic and no second launch, so it comes first; only when that leaves units idle long
// enough to pay for the merge launch are the keys split over workgroups as well.
// No two waves read the same key: nothing is shared, a wave waits for its own copies only and the key loop has no barrier.  K and V travel
// global -> LDS asynchronously; the K of the next block is requested when the scores of
// this one have been formed, its V when the products have.
//
// What bounds it, at head_dim 64 and one workgroup of 32 rows per compute unit: 2.05 us per 1000 keys, where the copies
// alone take 1.66 (64 bytes per clock and unit) and the arithmetic alone 2.0, 4.7 us of launch, first loads and merge, and 2.4 for
// a merge launch.  K fragments straight to registers (no LDS write and read): 3.6 us per 1000 keys, 32-byte pieces of a row per lane
// pair.  Four waves with the whole register file each: 5 to 6 us.  Against a grid of the longest user's tiles that began with 2000 cycles of
// decoding: one 2048 + 128 token request at 8/2 heads 10.2 -> 9.2 us per call; 8 requests of 512..4096 16.2 -> 14.0, with real-time
// tokens 16.2 -> 12.8; 4 of 8192 at head_dim 128 33.7 -> 29.2.  (The ordinary kernel: 18.0, 22.1, 25.0 and 37.6.)
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
template <int D, int RB, int NW, int SPS, int NST>
struct Serve {
    static constexpr int BLK = SUB * SPS;              // keys of a step
    static constexpr int TILE = BLK * D;               // elements of its K or V
    static constexpr int CPR = D / 8;                  // 16-byte chunks per row
    static constexpr int RPC = 64 / CPR;               // rows per 1 KB copy
    static constexpr int COPIES = BLK / RPC;           // copies of a step's K, and of its V
    static constexpr int ROWS = RB * SUB;              // packed rows of the workgroup
    static constexpr int Q_COPIES = ROWS / RPC;        // copies of their Q, dealt to the waves
    static constexpr int QUADS = D / 4, MERGED = SUB * QUADS;  // 4 features each, of a row block
    static constexpr int NIT = (MERGED + NW * 64 - 1) / (NW * 64);               // a thread's share of them
    static constexpr int PITCH = D + 4;                // floats per row of the merge buffer (16-byte words spread over the banks)
    // Registers: at head_dim 128 the O of two row blocks leaves no room for their Q, nor for their own keys, which are then requested behind
    // the key loop.
    static constexpr bool Q_IN_LDS = D == 128 && RB == 2;
    static_assert(!Q_IN_LDS || SPS == 1, "scores_of_lds");
    static constexpr int MERGE_BYTES = NW * SUB * (PITCH + 2) * 4;
    static constexpr int KV_BYTES = NW * NST * 2 * TILE * 2;
    static constexpr int Q = KV_BYTES, BEFORE = Q + ROWS * D * 2;
    static constexpr int BYTES = BEFORE > MERGE_BYTES ? BEFORE : MERGE_BYTES;
};
// what stands for a split that nobody writes: a NaN that no sum has, since no NaN of a bf16 input has these low bits
constexpr uint32_t NO_SPLIT = 0x7fc0d15cu;
__device__ inline float no_split() { return __uint_as_float(NO_SPLIT); }
__device__ inline bool is_no_split(float lse) { return __float_as_uint(lse) == NO_SPLIT; }
constexpr int UNITS = 256;   // compute units, each of which holds one workgroup
constexpr int GRID_TURN = 4;  // groups of tiles that take turns in a grid: the shader engines of an XCD
constexpr int TS_CAP = 512;  // real-time tokens of a user whose timestamps are searched in LDS

// How a launch's workgroups find their work.  An item is (user, kv head, head chunk, split, row tile); a user has as many as its lengths make.
// In a list the items of all users stand one after the other: every wave looks at all lengths, a lane to a user, and finds the item of its
// place by a running sum.  So a launch has no workgroups for tiles and splits that only the longest user has, and its XCDs have equally
// many whatever the lengths: XCD x takes a stretch of the list, or every eighth piece of `piece` items, whose row tiles read the same keys.
// For up to 64 users, and up to 192 where not all places of a grid have a unit at once; splits with the former only.
// In a grid a workgroup is a place of all (user, head, split, tile) that the bounds allow: many users even each other out, and a list would
// take every wave rounds of lanes, one trip to memory after the other.  (Target layers of 1 to 64 candidates, a list for all users against a grid for
// more than 64: 65..192 users with a unit for every place 1.05 to 1.09 of the grid's time, with up to two places per unit 0.96, with more 0.97
// to 1.02; 193..256 users 1.08 to 1.10, 385..512 1.15, more 1.18.)
struct ServeGrid {
    uint32_t piece;                   // 0: stretches
    uint32_t n_heads;                 // kv heads x head chunks
    uint32_t rows_magic;              // 2^32 / rows of a tile, rounded up (0: that is 1)
    int32_t n_splits;                 // the most that a user can have
    int32_t per;                      // blocks of keys of a piece in a list, if the longest user has as many as the bounds allow
};
inline uint32_t div_magic(uint32_t d) { return d == 1 ? 0u : (uint32_t)((1ull << 32) / d + 1); }
// n / d for n d < 2^32
__device__ inline uint32_t div_by(uint32_t n, uint32_t magic) { return magic == 0 ? n : __umulhi(n, magic); }
// n / d for n < 2^24
__device__ inline int div_small(int n, int d) {
    const int q = (int)((float)n * __builtin_amdgcn_rcpf((float)d)), r = n - q * d;
    return r < 0 ? q - 1 : r >= d ? q + 1 : q;
}
// the largest over all lanes, of numbers that are not negative
__device__ inline int max_of_lanes(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));  // row_shr 1, 2, 4, 8
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));  // row_bcast 15: into rows 1 and 3
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));  // row_bcast 31: into rows 2 and 3
    return __builtin_amdgcn_readlane(x, 63);
}
// sums over the lanes up to and with this one
__device__ inline int scan_lanes(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast 15: into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast 31: into rows 2 and 3
    return x;
}

// The arrays that the first loads go to and what finds the user stand alone at the front: arguments in scalar registers when the kernel
// starts (build.py, KERNARG_PRELOAD), while those inside Params take a load that costs 0.45 us at the start of a launch.
template <int D, int RB, int NW, int SPS, int NST, bool RT, bool PW, bool LIST>
__global__ __launch_bounds__(NW * 64, NW / 4) void serve_kernel(const int32_t* hist_len, const int32_t* n_targets, const int32_t* q_off,
                                                                const int32_t* kv_off, const int32_t* rt_len, int batch, int layer,
                                                                ServeGrid sg, Params p, RowMap map) {
    using SV = Serve<D, RB, NW, SPS, NST>;
    constexpr int BLK = SV::BLK, CP = SV::COPIES, QUADS = SV::QUADS, NIT = SV::NIT;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SV::BYTES];
    __shared__ __attribute__((aligned(256))) int ts_s[RT ? TS_CAP : 1], row_ts[RT ? SV::ROWS * 2 : 1];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    // (by the lengths, not by the call's bounds, which may be far above them; never more than there is room for)
    auto splits_of = [&](int blocks, int piece) __attribute__((always_inline)) { return min(max(1, div_small(blocks + piece - 1, piece)), sg.n_splits); };
    auto shortest_piece = [&](int blocks) __attribute__((always_inline)) { return max(div_small(blocks + sg.n_splits - 1, sg.n_splits), 1); };
    int L, T, R = 0, tile, gc, split = 0, n_live = 1, per = 0;  // per: blocks of keys of a piece
    int64_t q_base, kv_base;
    if constexpr (LIST) {
        struct Lane {  // a user's lengths, and its items with the keys in one piece
            int L, T, R, q, kv, tiles, in_one;
        };
        auto user_of_lane = [&](int first) __attribute__((always_inline)) {
            const int u = min(first + lane, batch - 1);
            Lane x = {hist_len[u], n_targets[u], RT ? rt_len[u] : 0, q_off[u], kv_off[u], 0, 0};
            x.tiles = (int)div_by((uint32_t)((layer == 0 ? x.L + x.R : 0) + x.T + map.rows - 1), sg.rows_magic);
            x.in_one = first + lane < batch ? x.tiles * (int)sg.n_heads : 0;
            return x;
        };
        Lane of = user_of_lane(0);
        const int blocks = (of.L + of.R + BLK - 1) / BLK;
        int items, splits = 1, upto, n_here, n_items;
        per = sg.per;
        auto cut = [&]() __attribute__((always_inline)) {
            if (sg.n_splits > 1) splits = splits_of(blocks, per);
            items = of.in_one * splits;
            upto = scan_lanes(items);
            n_here = __builtin_amdgcn_readlane(upto, 63);
        };
        cut();
        n_items = n_here;
        if (sg.n_splits > 1) {  // (64 users at most)
            // Pieces of the length that the longest user needs in order to have n_splits of them -- sg.per is that if the call's bounds are its
            // lengths, but they may be far above them -- or longer ones, until all items have a unit.
            if (__builtin_amdgcn_ballot_w64(splits == sg.n_splits) == 0) {
                per = shortest_piece(max_of_lanes(blocks));
                cut();
            }
            while (n_here > UNITS && __builtin_amdgcn_ballot_w64(splits > 1) != 0) {
                per += (per + 7) / 8;
                cut();
            }
            n_items = n_here;
        } else {
            for (int u = 64; u < batch; u += 64) n_items += __builtin_amdgcn_readlane(scan_lanes(user_of_lane(u).in_one), 63);
        }
        wait_vmem_loads();  // (all arrived with the first; the compiler may look for them behind the copies below, and would wait for those, too)
        const int xcd = blockIdx.x % N_XCD, slot_x = blockIdx.x / N_XCD;
        int at = sg.piece == 0 ? xcd * ((n_items + N_XCD - 1) / N_XCD) + slot_x
                               : ((slot_x / (int)sg.piece) * N_XCD + xcd) * (int)sg.piece + slot_x % (int)sg.piece;
        if (at >= n_items || (sg.piece == 0 && slot_x >= (n_items + N_XCD - 1) / N_XCD)) return;
        for (int u = 64; at >= n_here; u += 64) {
            at -= n_here;
            of = user_of_lane(u);
            items = of.in_one;
            upto = scan_lanes(items);
            n_here = __builtin_amdgcn_readlane(upto, 63);
            wait_vmem_loads();
        }
        const int u_lane = __builtin_popcountll(__builtin_amdgcn_ballot_w64(upto <= at));
        auto of_user = [&](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(x, u_lane); };
        at -= of_user(upto - items);
        const int n_tiles = of_user(of.tiles);
        L = of_user(of.L), T = of_user(of.T), n_live = of_user(splits);
        if (RT) R = of_user(of.R);
        q_base = of_user(of.q), kv_base = of_user(of.kv);
        const int ts_of = __builtin_amdgcn_readfirstlane(div_small(at, n_tiles));
        tile = at - ts_of * n_tiles;
        gc = sg.n_splits == 1 ? ts_of : __builtin_amdgcn_readfirstlane(div_small(ts_of, n_live));
        split = ts_of - gc * n_live;
    } else {
        const int xcd = blockIdx.x % N_XCD, slot_x = blockIdx.x / N_XCD, ny = (int)sg.n_heads * sg.n_splits;
        // A group is the tiles of a (user, head, split).  Four groups take turns, tile by tile and each time one place further: an XCD hands its workgroups
        // to its four shader engines in turn, and where most users have one tile of the two or four that the bounds allow the live ones would
        // all be two engines' or one's.  (Group after group, of 187 calls of 193 to 1000 users with bounds of four times the most
        // candidates 46 % took a tenth or more longer than in a list, up to twice; in turns 0.87 of the time, with true bounds 0.99.)
        const int four = __builtin_amdgcn_readfirstlane(div_small(slot_x / GRID_TURN, map.n_tiles));
        tile = slot_x / GRID_TURN - four * map.n_tiles;
        const int group = (four * GRID_TURN + ((slot_x - tile) & (GRID_TURN - 1))) * N_XCD + xcd;
        const int u = __builtin_amdgcn_readfirstlane(div_small(group, ny));
        if (u >= batch) return;
        L = hist_len[u], T = n_targets[u];
        if (RT) R = rt_len[u];
        q_base = q_off[u], kv_base = kv_off[u];
        gc = group - u * ny;
        if (sg.n_splits > 1) {
            const int blocks = (L + R + BLK - 1) / BLK, y = gc;
            gc = __builtin_amdgcn_readfirstlane(div_small(y, sg.n_splits));
            split = y - gc * sg.n_splits;
            per = shortest_piece(blocks);
            n_live = splits_of(blocks, per);
        }
        if (split >= n_live || tile * map.rows >= (layer == 0 ? L + R : 0) + T) return;
    }
    const int g = map.n_chunks == 1 ? gc : gc / map.n_chunks, chunk = gc - g * map.n_chunks;
    const int LK = L + R;  // keys that run through the tile loop: history, then real-time
    const int n_rows = layer == 0 ? LK + T : T;
    const int n_all = (LK + BLK - 1) / BLK, lo = split * per, hi = split == n_live - 1 ? n_all : lo + per;
    const PackedRows pr(map, tile, chunk, n_rows, g, p.Hq / p.Hkv);
    const int tok_shift = layer == 0 ? 0 : LK;  // token index of query row 0
    const int n_mine = max(hi - lo - wave + NW - 1, 0) / NW;  // steps of this wave: blocks lo + wave + i NW

    // K or V of step i to its slot.  Keys past the end repeat the last one (their weight is forced to zero).
    const __bf16* kg = (const __bf16*)p.k + (int64_t)g * D;
    const __bf16* vg = (const __bf16*)p.v + (int64_t)g * D;
    uint32_t voff[CP];  // byte offsets of the chunks this lane fetches from the first element of the block
#pragma unroll
    for (int j = 0; j < CP; j++) {
        const int trow = j * SV::RPC + lane / SV::CPR;
        voff[j] = (uint32_t)((trow * p.Hkv * D + ((lane % SV::CPR) ^ swizzle<D>(trow)) * 8) * 2);
    }
    auto slot = [&](int i) __attribute__((always_inline)) { return (wave * NST + (NST == 1 ? 0 : i % NST)) * (2 * SV::TILE * 2); };
    auto fetch = [&](const __bf16* src, int i, int part) __attribute__((always_inline)) {
        if (i >= n_mine) return;
        const int k0 = (lo + wave + i * NW) * BLK;
        const __bf16* base = src + (kv_base + k0) * p.Hkv * D;
        const uint32_t dst = lds_address(smem) + (uint32_t)(slot(i) + part * SV::TILE * 2);
        if (k0 + BLK <= LK) {
#pragma unroll
            for (int j = 0; j < CP; j++) copy16_global_to_lds_at(base, voff[j], dst + j * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < CP; j++) {
                const int trow = j * SV::RPC + lane / SV::CPR;
                const uint32_t past = (uint32_t)max(trow - (LK - 1 - k0), 0);
                copy16_global_to_lds_at(base, voff[j] - past * (uint32_t)(p.Hkv * D * 2), dst + j * 1024);
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
    auto request_own = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int it = 0; it < NIT; it++) {
                own_q[rb][it] = own_k[rb][it] = own_v[rb][it] = bf16x4{};
                if (split == 0) {
                    const int id = tid + it * NW * 64, c = id % QUADS, rl = id / QUADS;
                    const PackedRows::Row x = pr.at(rb * 32 + rl);
                    const uint32_t koff = (uint32_t)((x.row - pr.row0) * p.Hkv * D + 4 * c);
                    own_q[rb][it] = *(const bf16x4*)(q_tile + (uint32_t)(((x.row - pr.row0) * p.Hq + x.h) * D + 4 * c));
                    own_k[rb][it] = *(const bf16x4*)((const __bf16*)p.k + own_tile + koff);
                    own_v[rb][it] = *(const bf16x4*)((const __bf16*)p.v + own_tile + koff);
                }
            }
    };
    if constexpr (!SV::Q_IN_LDS) request_own();
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
    const __bf16* const q_rows = (const __bf16*)(smem + SV::Q);
    if constexpr (SV::Q_IN_LDS) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) rows.lim[rb] = L;
    } else {
        rows.take_q(q_rows, L);
    }
    if constexpr (RT) {
        // mask rule 2: the row sees the history and the real-time tokens strictly earlier than itself, a prefix
        const int32_t* ts = p.ts + kv_base + L;
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const int t = row_ts[rb * 64 + lane];
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
        const int k0 = (lo + wave + i * NW) * BLK, left = n_mine - 1 - i;
        // Two row blocks at head_dim 128 with limits per row: the fragment offsets of a masked step are formed in it, or they and the addresses made
        // of them would be kept across the loop (26 registers in scratch, reloaded in every step; without them 0.93 of the time on 785 requests in one piece, 0.97 on 483 in several).
        if constexpr (RT && TAIL && SV::Q_IN_LDS) {
            int l = lane;
            asm volatile("" : "+v"(l));
            rows.init_lane(p, l);
        }
        const __bf16* Ks = (const __bf16*)(smem + slot(i));
        floatx16 S[SPS][RB];
        wait_copies(min(NST - 1, left), true);  // newer than K_i: V_i and the following steps
        if constexpr (SV::Q_IN_LDS) {
            rows.scores_of_lds(S, Ks, q_rows);
        } else {
            rows.template scores<SPS>(S, Ks);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // K_i has been read
        fetch(kg, i + NST, 0);
        wait_copies(min(NST - 1, left), left >= NST);  // newer than V_i: the following steps, and K_(i + NST)
        rows.template absorb<TAIL, SPS>(S, Ks + SV::TILE, LK - k0, k0, L, i == 0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fetch(vg, i + NST, 1);
    };
    // blocks of history keys first, then those that need a mask (the last one; more with real-time tokens)
    const int n_whole = min(max(min(hi, L / BLK) - lo - wave + NW - 1, 0) / NW, n_mine);
    for (int i = 0; i < n_whole; i++) step(i, std::false_type{});
    for (int i = n_whole; i < n_mine; i++) step(i, std::true_type{});

    if constexpr (SV::Q_IN_LDS) request_own();
    // ---- the own keys' logits, summed over the threads of a row: log2 units (PW: the weight itself), -inf (0) where there is none
    float own[RB][NIT];
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int rl = (tid + it * NW * 64) / QUADS;
            const bool has = split == 0 && tok_shift + pr.at(rb * 32 + rl).row >= L;
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
        const int c = id % QUADS, l = id / QUADS;  // 4 features of a row
        const PackedRows::Row x = pr.at(rb * 32 + l);
        float mx = PW ? 0.f : fmaxf(own[rb][it], -1e30f);
        float2 ml[NW];
        if constexpr (!PW) {
#pragma unroll
            for (int k = 0; k < NW; k++) {
                ml[k] = *(const float2*)(stat + (k * SUB + l) * 2);
                mx = fmaxf(mx, ml[k].x);
            }
        }
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
        float sum = 0.f;
        if (split == 0 && tok_shift + x.row >= L) {  // (by the row, not by the logit: one that is NaN has to show)
            const float f = PW ? own[rb][it] : fast_exp2(own[rb][it] - mx);
            sum = f;
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = f * (float)own_v[rb][it][j];
        }
#pragma unroll
        for (int k = 0; k < NW; k++) {
            const float f = PW ? 1.f : fast_exp2(ml[k].x - mx);  // 0 for a wave that saw no key
            const floatx4 ok = *(const floatx4*)(acc + (k * SUB + l) * SV::PITCH + 4 * c);
            if constexpr (!PW) sum = fmaf(f, ml[k].y, sum);
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = fmaf(f, ok[j], o[j]);
        }
        if (!x.live || id >= SV::MERGED) continue;
        const float inv = PW ? p.norm * p.scale : (sum > 0.f ? 1.f / sum : 0.f);
        const float lse = sum > 0.f ? (mx + __builtin_amdgcn_logf(sum)) * LN2 : sum == sum ? -INFINITY : sum;  // (NaN shows here, too)
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
            *(floatx4*)((float*)p.out + (((int64_t)split * p.total_q + row) * p.Hq + x.h) * D + 4 * c) = o4;
            if (c == 0) p.lse[((int64_t)split * p.Hq + x.h) * p.total_q + row] = PW ? 0.f : lse;
            // the splits that this user's keys do not reach are nobody's: nothing was left there
            if (c == 0 && split == 0)
                for (int k = n_live; k < sg.n_splits; k++) p.lse[((int64_t)k * p.Hq + x.h) * p.total_q + row] = no_split();
        }
    }
    });
}

// out = sum_s w_s O_s / sum_s w_s with w_s = exp(lse_s - max lse), lse = max lse + log sum_s w_s: the exact
// combination of softmax results over disjoint key sets.  One thread per 4 features of a (row, head).
// PW: the partial results are partial sums of non-normalised weights: out = sum_s O_s, no lse.
// All loads of a thread travel together, AT_ONCE splits of them: one trip to memory is most of what this launch takes.  (Split after split,
// as the remainder of an unrolled loop is: 2 us more for 4 splits.)  The splits that a user's keys do not reach are the last ones, and
// marked: a launch has as many as the longest user may need, and one with bounds far above its lengths more than any has.  MORE: than AT_ONCE
// (a look at the mark behind them costs 0.1 us where there is none).
template <int D, int AT_ONCE, bool MORE, bool PW>
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
            ls[s] = lse_part[at_lse + i * l_stride];
            os[s] = *(const floatx4*)(o_part + id * 4 + i * o_stride);
        }
        const float next = MORE ? lse_part[at_lse + min(s0 + AT_ONCE, n_splits - 1) * l_stride] : 0.f;
        const float before = mx;
        if constexpr (!PW) {
#pragma unroll
            for (int s = 0; s < AT_ONCE; s++) mx = fmaxf(mx, ls[s]);  // (the mark is a NaN)
            const float f = before > -INFINITY ? __expf(before - mx) : 0.f;
            sum *= f;
            o *= f;
        }
#pragma unroll
        for (int s = 0; s < AT_ONCE; s++) {
            const bool none = s0 + s >= n_splits || is_no_split(ls[s]);
            const float w = none ? 0.f : PW ? 1.f : __expf(ls[s] - mx);
            sum += w;
#pragma unroll
            for (int j = 0; j < 4; j++) o[j] = none || ls[s] == -INFINITY ? o[j] : fmaf(w, os[s][j], o[j]);  // (-inf: no key that the row sees)
        }
        if (!MORE || is_no_split(next)) break;
    }
    const float inv = PW ? 1.f : 1.f / sum;
    bf16x4 o4;
#pragma unroll
    for (int j = 0; j < 4; j++) o4[j] = (__bf16)(o[j] * inv);
    *(bf16x4*)((__bf16*)out + id * 4) = o4;
    if (!PW && id % QUADS == 0) lse[at_lse] = mx + __logf(sum);
}

// the most row tiles x kv heads x head chunks that a call's users can have, whatever their lengths
int64_t most_tiles(const Params& p, const RowMap& map) {
    const int64_t by_rows = (p.total_q + (int64_t)p.batch * (map.rows - 1)) / map.rows;
    return std::min(by_rows, (int64_t)p.batch * map.n_tiles) * p.Hkv * map.n_chunks;
}

// (user, kv head, head chunk), and the places of a grid: tiles that they have by the bounds
int64_t groups_of(const Params& p, const RowMap& map) { return (int64_t)p.batch * p.Hkv * map.n_chunks; }
int64_t places(const Params& p, const RowMap& map) { return groups_of(p, map) * map.n_tiles; }
// A list or a grid: see ServeGrid.
bool takes_list(const Params& p, const RowMap& map) { return p.batch <= 64 || (p.batch <= 192 && places(p, map) > UNITS); }

template <int D, int RB, int NW, int SPS, int NST, bool LIST>
auto kernel_of(const Params& p) {
    if (p.pointwise) return p.rt_len ? serve_kernel<D, RB, NW, SPS, NST, true, true, LIST> : serve_kernel<D, RB, NW, SPS, NST, false, true, LIST>;
    return p.rt_len ? serve_kernel<D, RB, NW, SPS, NST, true, false, LIST> : serve_kernel<D, RB, NW, SPS, NST, false, false, LIST>;
}

template <int D, bool PW>
auto merge_of(int n_splits) {
    return n_splits <= 2 ? merge_splits_kernel<D, 2, false, PW> : n_splits <= 4 ? merge_splits_kernel<D, 4, false, PW>
         : n_splits <= 8 ? merge_splits_kernel<D, 8, false, PW> : merge_splits_kernel<D, 8, true, PW>;
}

template <int D, int RB, int NW, int SPS, int NST>
hipError_t launch(const Params& p, hipStream_t s) {
    const int64_t rows = max_query_rows(p);
    if (rows <= 0) return hipSuccess;
    const RowMap map = row_map(RB * 32, p.Hq, p.Hkv, rows);
    const int64_t max_blocks = (most_keys(p) + SUB * SPS - 1) / (SUB * SPS);
    ServeGrid sg;
    sg.per = (int32_t)std::max<int64_t>((max_blocks + p.n_splits - 1) / p.n_splits, 1);
    sg.n_splits = (int32_t)std::max<int64_t>((max_blocks + sg.per - 1) / sg.per, 1);
    sg.n_heads = (uint32_t)(p.Hkv * map.n_chunks);
    sg.rows_magic = div_magic((uint32_t)map.rows);
    const int64_t tiles = most_tiles(p, map), most = std::min(tiles * sg.n_splits, std::max<int64_t>(tiles, UNITS));
    sg.piece = most <= 320 ? 0 : 4;
    const int64_t dealt = N_XCD * (sg.piece == 0 ? 1 : sg.piece);
    const bool list = takes_list(p, map);
    constexpr int64_t turn = N_XCD * GRID_TURN;
    const int64_t n_blocks = list ? (most + dealt - 1) / dealt * dealt : work_grid((groups_of(p, map) * sg.n_splits + turn - 1) / turn * turn, map.n_tiles);
    // Partial results through the same pointers as results: with two more of them the form with real-time tokens runs out of scalar registers
    // and waits for loads at its start (8 requests of 512..4096 keys 13.11 -> 12.72 us).
    Params to = p;
    if (sg.n_splits > 1) to.out = p.o_part, to.lse = p.lse_part;
    auto kernel = list ? kernel_of<D, RB, NW, SPS, NST, true>(p) : kernel_of<D, RB, NW, SPS, NST, false>(p);
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_blocks), dim3(NW * 64), 0, s, p.hist_len, p.n_targets, p.q_off, p.kv_off, p.rt_len, p.batch, p.layer,
                       sg, to, map);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || sg.n_splits == 1) return e;
    const int64_t threads = p.total_q * p.Hq * (p.d / 4);
    const int n = (int)sg.n_splits;
    auto merge = p.pointwise ? merge_of<D, true>(n) : merge_of<D, false>(n);
    hipLaunchKernelGGL(merge, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       p.o_part, p.lse_part, p.total_q, p.Hq, n, p.out, p.lse);
    return hipGetLastError();
}

// workgroups with work to do: `lanes` packed rows each, from the bounds and the number of query rows of the call
int64_t live_tiles(const Params& p, int lanes) {
    const RowMap map = row_map(lanes, p.Hq, p.Hkv, max_query_rows(p));
    const int64_t groups = groups_of(p, map);
    return std::min(groups * map.n_tiles, p.total_q * p.Hkv * map.n_chunks / map.rows + groups / 2);
}

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

// Estimated times of a call (us), from fits of 8775 calls timed in every form (1 to 64 users, target layers of 2 to 300 candidates and, a
// third of the calls, full layers; 64 to 16384 keys, all of one length or spread over a factor of 8; with and without real-time tokens and
// with pointwise weights; inputs of four calls in turn).
//
// The ordinary kernel, up to two workgroups per unit: the longest one, more the fuller the chip, and the schedule's launch.
static double ordinary_us(const Params& p, int64_t workgroups) {
    struct { double launch, schedule, key, key_full, second; } c;
    if (p.d == 32) c = {3.6, 2.6, 9.3e-3, 5.9e-3, 1.9};
    else if (p.d == 128) c = {7.5, 1.9, 17.e-3, 8.3e-3, 13.};
    else if (fwd_workgroup_rows(p) == 128) c = {5.2, 2.6, 12.e-3, 11.e-3, 2.8};
    else c = {6.7, 1.1, 13.e-3, 17.e-3, 7.4};
    const double fill = workgroups / (double)UNITS;
    return c.launch + (forward_needs_schedule(p) ? c.schedule : 0.) + c.key * longest_keys(p) + c.key_full * mean_keys(p) * fill + c.second * std::max(0., fill - 1.);
}
// The kernel above, `row_blocks` blocks of 32 rows per workgroup and the keys of the longest user in `splits` pieces.  One workgroup per unit; a
// key costs more the fuller the chip (its XCDs' L2s feed all units).  In one piece, more items than units take rounds, whole ones where
// all have the same keys.  In several, the pieces are as long as it takes for all items to have a unit, and the merge costs a launch and
// the partial results.
struct ServeSize {
    double longest, mean, part;  // keys of the longest user and of the mean; MB of a partial result
    double items[2];             // workgroups with keys in one piece, of one and two row blocks
    ServeSize(const Params& p)
        : longest(longest_keys(p)), mean(mean_keys(p)), part(1e-6 * p.total_q * p.Hq * p.d * 4), items{(double)live_tiles(p, 32), (double)live_tiles(p, 64)} {}
};
static double serve_us(const Params& p, const ServeSize& size, int row_blocks, int splits) {
    struct { double launch, item, key, key_full, jagged, merge, part, rt, piece, partial; } c;
    if (p.d == 32) c = {-0.46, 4.6, 2.2, 1.0, 0.43, 2.4, 0.55, 0.48, 0.34, 0.23};
    else if (p.d == 64 && row_blocks == 1) c = {0.85, 3.8, 2.6, 1.3, 0.66, 2.4, 0.35, 0.49, 0.38, 0.18};
    else if (p.d == 64) c = {0.89, 5.4, 4.0, 1.7, 0.78, 2.5, 0.35, 0.96, 0.37, 0.13};
    else if (row_blocks == 1) c = {0.93, 4.9, 5.0, 1.9, 0.77, 2.3, 0.19, 0.41, 0.51, 0.15};
    else c = {-0.34, 9.3, 5.9, 3.5, 0.73, 2.6, 0.22, 2.2, 0.45, 0.14};
    const double longest = size.longest, mean = size.mean, items = size.items[row_blocks - 1], rounds = items / UNITS;
    const bool even = mean > 0.9 * longest;
    // (more than 64 users: 1.2 to 1.45 times what the fits say, by 1400 target layers of 65 to 1024; with this factor the chosen form takes 1.03 of
    // the best one's time)
    const double fixed = c.launch + (p.rt_len ? c.rt : 0.), grid = p.batch > 64 ? 1.25 : 1.;
    double keys = longest, pieces = items;
    if (splits > 1) {
        const double fits = p.batch > 64 ? 0. : items < 250. ? items * mean / std::max(UNITS - c.piece * items, 16.) : longest;
        keys = std::min(std::max(longest / splits, fits), longest);
        const double of_mean = mean / std::max(keys, 1.);
        pieces = items * (even ? std::ceil(of_mean - 0.01) : of_mean + c.piece);
    }
    const double key = 1e-3 * (c.key + c.key_full * std::min(1., pieces / UNITS));
    const double whole = std::ceil(rounds);
    const double many = (even ? whole + c.partial * (rounds - whole) : rounds + c.jagged) * (c.item + key * mean);
    if (splits == 1) return grid * (fixed + (rounds <= 1. ? c.item + key * longest : std::max(c.item + key * longest, many)));
    return grid * (fixed + c.merge + c.part * splits * size.part + (rounds <= 1. ? c.item + key * keys : std::max(c.item + key * longest, many)));
}

// What a call takes: this kernel with one or two row blocks per workgroup and the keys in up to `room` pieces, or the ordinary one,
// which shares each K/V tile among 128 or 256 rows and keeps two workgroups on a unit.  By the estimates above, of which against the best
// form of each call 1.2 % of the time are lost on target layers (of 6060, 762 lose 3 % or more and 203 a tenth) and 0.6 on full ones.  The
// rule before, with a line at 256 workgroups of 32 rows and the merge at 4.2 us, lost 5.7 % on the former, and a tenth or more in 1262.
struct ServeForm {
    int row_blocks, splits;  // splits 0: the ordinary kernel
};
static ServeForm serve_form(const Params& p, int room) {
    const int64_t ordinary = live_tiles(p, fwd_workgroup_rows(p)), blocks = most_keys(p) / SUB;
    const int64_t in_grid = p.batch <= 64 ? 0 : places(p, row_map(32, p.Hq, p.Hkv, max_query_rows(p)));
    if (ordinary >= 512 || p.batch > 1024 || max_query_rows(p) >= 1 << 20 || in_grid >= 1 << 24) return {1, 0};
    ServeForm best = {1, 0};
    double best_us = ordinary_us(p, ordinary);
    const ServeSize size(p);
    for (int splits : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
        if (splits > 1 && (splits > room || splits > blocks / 6 || blocks >= 1 << 15 || in_grid * splits > UNITS)) break;
        for (int rb = 1; rb <= (p.d == 32 ? 1 : 2); rb++) {
            const double us = serve_us(p, size, rb, splits);
            if (us < best_us) best_us = us, best = {rb, splits};
        }
    }
    return best;
}
int serve_splits(const Params& p, int room) { return serve_form(p, room).splits; }
// (of the same estimates, once the splits are chosen)
int serve_row_blocks(const Params& p) {
    const ServeSize size(p);
    return p.d != 32 && serve_us(p, size, 2, p.n_splits) < serve_us(p, size, 1, p.n_splits) ? 2 : 1;
}

bool serve_takes_list(const Params& p) { return takes_list(p, row_map(serve_row_blocks(p) * 32, p.Hq, p.Hkv, max_query_rows(p))); }

hipError_t launch_serve_bf16(const Params& p, hipStream_t s) {
    const bool two = serve_row_blocks(p) == 2;
    // short lists of keys per wave: single sub-tiles divide more evenly than pairs
    const bool brief = (int64_t)longest_keys(p) / p.n_splits <= 1024;
    hipError_t e;
    timing_begin(MTFM_HTA_KERNEL_FWD, s);
    switch (p.d) {
        case 32: e = launch<32, 1, 8, 2, 2>(p, s); break;
        case 64: e = two ? launch<64, 2, 8, 1, 2>(p, s) : brief ? launch<64, 1, 8, 1, 2>(p, s) : launch<64, 1, 8, 2, 1>(p, s); break;
        case 128: e = two ? launch<128, 2, 8, 1, 1>(p, s) : launch<128, 1, 8, 1, 1>(p, s); break;
        default: e = hipErrorInvalidValue;
    }
    timing_end(MTFM_HTA_KERNEL_FWD, s);
    return e;
}

}  // namespace hta
