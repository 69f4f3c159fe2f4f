// bf16 backward of Hybrid Target Attention for gfx950 in one pass (head_dim 64, users of at most 512 packed (row, query head) pairs
// per kv head: the candidates of a target-only layer): S, dP and the weights of every (row, key) pair are formed once and feed dQ, dK
// and dV -- five matrix products per pair, where a dQ pass and a dK/dV pass of their own (hta_bwd_bf16.hip) need seven and form every
// weight twice.
//
// A workgroup takes a (user, kv head) whole: no gradient ever crosses a workgroup, so there are no atomics and every sum has a fixed
// order.  Its waves hold the user's pairs, two units of 32 each, and walk the keys in blocks of 32:
//   phase 1  a wave forms S^T = K Q^T, dP^T = V dO^T, P and dS of its units (row on the lane, as in the dQ pass), adds
//            dQ^T += K^T dS^T straight from the registers and leaves P and dS as bf16 in LDS, [row][key];
//   phase 2  dK^T[d][key] = Q^T dS and dV^T = dO^T P contract over the rows: P and dS come back through the transposed LDS read
//            with the key on the lane, against Q^T and dO^T, which never change: wave t of four holds one 32-wide half of the features
//            of dO (t = 0, 1) or Q (t = 2, 3), of the first units in registers, of the second ones it reads them from LDS.
// One barrier behind each phase.  What fits decides the shape: dQ, Q, dO and the operands of phase 2 of 512 pairs are 384 KB, so the
// second units' Q and dO rest in LDS, where both phases read them (all in registers left none to fetch operands ahead with: 3.5 ms
// on 512 users x 2048 keys x 128 candidates, 16/4 heads, against 1.6).  Up to 256 pairs a workgroup is one group of four waves
// and a compute unit holds two, whose barriers do not meet; above, two groups share the K/V tiles and exchange their sums of phase 2
// (16 KB per block) so that each finishes half of it.  (Two groups half a block apart, one's matrix products next to the other's
// exponentials, took as long as in step; so did S of the next block formed in phase 2.)
// Backward calls back to back, two passes -> this one, in turn on one box: that workload 2.09 -> 1.63 ms; 600 users x 1000 keys x 60, 8/2
// heads 399 -> 269 us.  Bound by
// the sum of matrix and vector work: a SIMD is busy with 2560 cycles of products and 2500 of vector instructions per block of 16
// units, of about 5200.  (Users of more pairs, taken 512 at a time with float32 dK, dV resting in memory in between, were no faster
// than two passes: 1.52 against 1.39 ms on a full layer of 256 users x 512..1024 keys.)
// dk/dv of a target token's own key come from the lanes that hold its rows, in the prologue.
#include "../../include/mtfm_hta.h"
#include "../../include/mtfm_hta_timing.h"
#include "hta_common.h"
#include "hta_mfma.h"
#include "hta_rows.h"
#include "hta_tiles.h"

#include <algorithm>
#include <cmath>

namespace hta {
namespace {

constexpr int OP_D = 64;                // head_dim
constexpr int OP_TILE = 32 * OP_D * 2;  // bytes of a 32-row tile
constexpr int OP_UNIT = 32 * 32 * 2;    // bytes of a unit's P (or dS) block, [row][key] bf16
constexpr int OP_SUMS = 4 * 4096;       // bytes of a block's dV, dK (two halves of the features each) in float32
// A workgroup of NG groups of four waves: packed pairs of a user, byte offsets in LDS.  P and dS of the units; Q and dO of the second
// units; sums that the groups exchange; K/V.  (Q and dO of the first units are where P and dS go while phase 2's operands are
// taken from them.)
template <int NG>
struct OnePass {
    static constexpr int NW = 4 * NG, LANES = 256 * NG;
    static constexpr int P = 0, DS = 8 * NG * OP_UNIT, ROWS0 = 0, ROWS1 = 16 * NG * OP_UNIT, DO = NW * OP_TILE;  // (DO: dO behind Q)
    static constexpr int X = ROWS1 + 2 * NW * OP_TILE, KV = X + (NG > 1 ? OP_SUMS : 0), STAGE = 2 * OP_TILE;
    static constexpr int BYTES = KV + 2 * STAGE;
    static_assert(BYTES * (NG > 1 ? 1 : 2) == 160 * 1024, "LDS");
};

constexpr int OP_MAX_HEADS = 8;
// Blocks before an item's end at which the workgroup takes its next item.  Wave 0 waits for the answer where it asks, and the others at the next barrier.
// (Left in flight until behind the blocks, in a register of its own: eight calls of 300 to 700 users 1.003 of the time, 1.005 to 1.014 where there are two
// groups of waves, 136 shorter calls 1.002.)  Asked for with the item's start, the last items of the lists wait behind items in progress while other
// workgroups leave; asked for later is not better, either: three blocks before the end 562 users of 55..444 keys, 8/1 heads, pointwise 49.5 -> 56.1 us, 306
// of 130..521, 8/2, 60.6 -> 68.0.  Whole steps, asked for with the start -> here: 227 users of 318..1275 keys, 8/2 heads, 240 -> 207 us, 131 of 289..1157,
// 16/4, 137 -> 126, 453 of 178..1429, 4/4, 368 -> 354, 96 of 82..658, 16/4, pointwise 111 -> 87; 160 target layers at random 0.988 of the time, 22 of them
// below 0.97 and four above 1.02 (1.04 at most).
// An item of fewer blocks asks as soon as its lengths are read, and where that is the mean item all do with their start, before that: by the mean, which
// does not follow the bounds of a call.  (By the bounds, that is late in calls of short users with roomy bounds: 463 users of 39..156 keys, 8/2 heads,
// 46.6 -> 48.4 us, 56 calls of 64 to 160 keys in the mean with bounds of four times the longest 1.010.  With true bounds 24 calls of more keys in the
// mean 1.019 if all ask with their start, 24 of 94 to 160 1.001.)
constexpr int ASK_AHEAD = 6;
template <int NG, bool RT, bool PW>
__global__ __launch_bounds__(NG * 256, 2) void bwd_onepass_kernel(Params p, RowMap map, unsigned per_xcd, bool ask_late) {
    using OP = OnePass<NG>;
    constexpr int D = OP_D, NKS = D / 16, NDB = D / 32, NW = OP::NW;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[OP::BYTES];
    int* const s_item = (int*)(smem + OP::KV);  // (between two items nothing rests there)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = NG > 1 ? wave >> 2 : 0, t = wave & 3;
    const int r = p.Hq / p.Hkv;
    const float c2 = p.scale * LOG2E, neg_c2 = -c2;
    const __bf16* const kg = (const __bf16*)p.k;
    const __bf16* const vg = (const __bf16*)p.v;
    const uint32_t lds0 = lds_address(smem);

    auto at = [&](int byte) __attribute__((always_inline)) { return (__bf16*)(smem + byte); };
    // a: address of the fragment's first piece.  (Offsets of whole KB leave the low bits alone, so the XORs of the swizzles apply
    // to finished addresses.)
    auto tr64 = [&](int a, int plus) __attribute__((always_inline)) { return lds_read_tr_pair(at(a + plus), at((a ^ 32) + plus + 1024)); };
    // An address formed here is formed anew in every block: kept from the loop's start, the XORed ones would take up the
    // registers that the loop is short of.
    auto fresh = [](int x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    // (Lane arithmetic is done where it is needed, for the same reason: the compiler would keep all of it, from the start of the kernel.)
    auto lane_anew = []() __attribute__((always_inline)) {  // the lane's index, likewise
        int x;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
        return x;
    };

    const int xcd = blockIdx.x % N_XCD;
    unsigned taken = blockIdx.x / N_XCD;
    // takes the next item: once per item, at one of three places
    auto ask = [&]() __attribute__((always_inline)) {
        if (tid == 0) taken = queue_take_ahead(p.queue, xcd, per_xcd, gridDim.x);
    };

    auto process = [&](unsigned id) {
        const WorkItem w = decode_work(id, p.batch * p.Hkv, p.Hkv, 1);
        if (!ask_late || !w.valid) ask();
        if (!w.valid) return;
        // (uniform values, which the compiler cannot tell of loads in a loop that also stores)
        auto uniform = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
        auto uniform64 = [&](int64_t x) __attribute__((always_inline)) {
            return (int64_t)((uint64_t)(uint32_t)uniform((int)(x >> 32)) << 32 | (uint32_t)uniform((int)x));
        };
        const int b = uniform(scheduled_user(p, w.user_slot)), g = w.y;
        const int L = uniform(p.hist_len[b]), T = uniform(p.n_targets[b]);
        const int LK = L + (RT ? uniform(p.rt_len[b]) : 0);  // keys of the block loop: history, then real-time
        const int n_rows = p.layer == 0 ? LK + T : T, tok_shift = p.layer == 0 ? 0 : LK;
        const int64_t q_base = uniform(p.q_off[b]), kv_base = uniform(p.kv_off[b]);
        const int n_blocks = (LK + 31) / 32;
        if (ask_late && (n_blocks < ASK_AHEAD || n_rows == 0)) ask();
        if (n_rows == 0) {  // nobody attends to these keys: dk = dv = 0
            const bf16x8 zero = {};
            for (int i = tid; i < LK * (D / 8); i += NW * 64) {
                const int64_t off = ((kv_base + i / (D / 8)) * p.Hkv + g) * D + i % (D / 8) * 8;
                *(bf16x8*)((__bf16*)p.dk + off) = zero;
                *(bf16x8*)((__bf16*)p.dv + off) = zero;
            }
            return;
        }
        // K/V copies: wave t of a group brings rows 8 t .. of a tile, of K group 0, of V the last one
        auto issue_kv = [&](int i) __attribute__((always_inline)) {
            const uint32_t dst = lds0 + OP::KV + (uint32_t)(i & 1) * OP::STAGE + (uint32_t)t * 1024u;
            const int64_t base = uniform64(((kv_base + 32 * (int64_t)i) * p.Hkv + g) * D);
            const int x = lane_anew(), crow = 8 * t + (x >> 3);
            const int row = min(crow, LK - 1 - 32 * i);  // keys past the end repeat the last one: finite data whose weights are set to zero
            const uint32_t voff = (uint32_t)((row * p.Hkv * D + (((x & 7) ^ swizzle<64>(crow)) << 3)) * 2);
            if (group == 0) copy16_global_to_lds_at(kg + base, voff, dst);
            if (group == NG - 1) copy16_global_to_lds_at(vg + base, voff, dst + OP_TILE);
        };

        const int lane = lane_anew(), l32 = lane & 31, hf = lane >> 5;
        // per-lane byte offsets, from which the others follow by XOR of constants (swizzles: hta_mfma.h)
        const int trow = 4 * hf + ((lane & 15) >> 2), tchunk = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
        const int nat0 = l32 * 128 + ((hf ^ swizzle<64>(l32)) << 4);                              // row l32, chunk hf       of a 64-wide tile
        const int tr0 = trow * 128 + ((tchunk ^ swizzle<64>(trow)) << 4) + 8 * (lane & 1);        // transposed fragment     of a 64-wide tile
        // P, dS: row l32, keys 4 hf .. of chunk 0.  The 8-byte halves of a chunk are exchanged in every second pair of rows: a store
        // takes 16 lanes at a time and then finds each of 16 rows on banks of its own.
        auto pw0 = [&]() __attribute__((always_inline)) {
            const int ln = lane_anew(), row = ln & 31;
            return row * 64 + (swizzle<32>(row) << 4) + 8 * ((ln >> 5) ^ ((row >> 1) & 1));
        };
        const int pr0 = trow * 64 + ((tchunk ^ swizzle<32>(trow)) << 4) + 8 * ((lane & 1) ^ ((trow >> 1) & 1));
        const PackedRows pr(map, 0, 0, n_rows, g, r);  // (rows beyond the caller's bound on them would be left out)
        const int n_units = (min(n_rows, map.rows) * map.heads + 31) / 32;
        if (n_blocks > 0) issue_kv(0);
        // ---- the rows of this wave: units wave and wave + NW; all that the two need is requested before any of it is used
        bf16x8 q0[NKS], do0[NKS];  // of the first unit; the second one's stay in LDS
        floatx16 dQ[2][NDB];       // dQ^T: [d (registers)][row (lanes)]
        float lse2[2], dl[2];
        int lim[2], own[2];        // RT: leading keys that the lane's row sees, and its own key among the real-time ones
        {
            const bf16x8 zero = {};
            bf16x8 ox[2][NKS], kk[2][NKS], vv[2][NKS];
            bool targets[2];     // uniform: are there target rows in the unit
            float fk[2], fv[2];  // weights of a target row in the dk, dv of its own key
            // Q and dO straight to LDS, where the wave finds its own rows (and the transposed operands of phase 2 come from):
            // copy j brings rows 8 j .. of a tile.  No branches here: a lane or unit that stands for no row repeats the last one.
#pragma unroll
            for (int s = 0; s < 2; s++) {
                const int pos = (s == 0 ? OP::ROWS0 : OP::ROWS1) + wave * OP_TILE;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int crow = 8 * j + (lane >> 3);
                    const PackedRows::Row x = pr.at((NW * s + wave) * 32 + crow);
                    const int64_t off = ((q_base + x.row) * p.Hq + x.h) * D + (((lane & 7) ^ swizzle<64>(crow)) << 3);
                    copy16_global_to_lds_at((const __bf16*)p.q + off, lds0 + (uint32_t)(pos + j * 1024));
                    copy16_global_to_lds_at((const __bf16*)p.dout + off, lds0 + (uint32_t)(pos + OP::DO + j * 1024));
                }
            }
#pragma unroll
            for (int s = 0; s < 2; s++) {
                const PackedRows::Row x = pr.at((NW * s + wave) * 32 + l32);
                const int64_t off = ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
                const int64_t koff = ((kv_base + tok_shift + x.row) * p.Hkv + g) * D + 8 * hf;
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    if constexpr (!PW) ox[s][ks] = *(const bf16x8*)((const __bf16*)p.out + off + ks * 16);
                    kk[s][ks] = *(const bf16x8*)(kg + koff + ks * 16);
                    vv[s][ks] = *(const bf16x8*)(vg + koff + ks * 16);
                }
                lse2[s] = PW ? 0.f : p.lse[(int64_t)x.h * p.total_q + q_base + x.row];
                lim[s] = RT ? p.lim[q_base + x.row] : L;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int s = 0; s < 2; s++) {
                const PackedRows::Row x = pr.at((NW * s + wave) * 32 + l32);
                const int pos = (s == 0 ? OP::ROWS0 : OP::ROWS1) + wave * OP_TILE;
                // a lane that stands for no row adds nothing anywhere: its Q and dO are zeros, and so are its weights
                const int tok = tok_shift + x.row;
                const bool has_own = tok >= L && x.live;  // a target or real-time row sees its own key, where its dQ starts
                bf16x8 qx[NKS], dox[NKS];
                float part = 0.f, sp = 0.f, dpp = 0.f;
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    qx[ks] = *(const bf16x8*)at(pos + (nat0 ^ (ks << 5)));
                    dox[ks] = *(const bf16x8*)at(pos + OP::DO + (nat0 ^ (ks << 5)));
                    qx[ks] = x.live ? qx[ks] : zero;
                    dox[ks] = x.live ? dox[ks] : zero;
                    kk[s][ks] = has_own ? kk[s][ks] : zero;
                    vv[s][ks] = has_own ? vv[s][ks] : zero;
                    if (s == 0) q0[ks] = qx[ks], do0[ks] = dox[ks];
                    if constexpr (!PW) part = dot_bf16x8(part, dox[ks], x.live ? ox[s][ks] : zero);
                    sp = dot_bf16x8(sp, qx[ks], kk[s][ks]);
                    dpp = dot_bf16x8(dpp, dox[ks], vv[s][ks]);
                    *(bf16x8*)at(pos + (nat0 ^ (ks << 5))) = qx[ks];
                    *(bf16x8*)at(pos + OP::DO + (nat0 ^ (ks << 5))) = dox[ks];
                }
                sp += other_half(sp);
                dpp += other_half(dpp);
                lse2[s] = x.live ? lse2[s] * LOG2E : INFINITY;
                dl[s] = PW ? 0.f : -(part + other_half(part));
                own[s] = RT && has_own && tok < LK ? tok : -1;
                float pw, ds;
                if constexpr (PW) {
                    const float sg = pw_sigmoid(sp, neg_c2);
                    pw = pw_silu(sp, sg);  // P / scale, here and below
                    ds = dpp * pw_silu_prime_of(pw, sg, p.scale);
                } else {
                    pw = fast_exp2(fmaf(sp, c2, -lse2[s]));
                    ds = pw * (dpp + dl[s]);
                }
                if (!has_own) ds = pw = 0.f;
                // K of the key with the features where dQ has them: registers 4 v4 .. hold 8 v4 + 4 hf .. of 32
                static_for<0, NKS>([&](auto Ks) {
                    constexpr int ks = decltype(Ks)::value;
                    typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
                    const uintx4 k4 = __builtin_bit_cast(uintx4, kk[s][ks]);
                    const auto e0 = __builtin_amdgcn_permlane32_swap(k4[0], k4[2], false, false);
                    const auto e1 = __builtin_amdgcn_permlane32_swap(k4[1], k4[3], false, false);
                    const uintx4 d4 = {(unsigned)e0[0], (unsigned)e1[0], (unsigned)e0[1], (unsigned)e1[1]};
                    const bf16x8 kd = __builtin_bit_cast(bf16x8, d4);
#pragma unroll
                    for (int j = 0; j < 8; j++) dQ[s][ks / 2][8 * (ks % 2) + j] = ds * (float)kd[j];
                });
                const bool target = has_own && tok >= LK;
                fk[s] = !target ? 0.f : PW ? ds * p.scale * p.norm : ds * p.scale;
                fv[s] = !target ? 0.f : PW ? pw * p.scale * p.norm : pw;
                targets[s] = __builtin_amdgcn_ballot_w64(target) != 0;
                __builtin_amdgcn_sched_barrier(0);
            }
            // A target's key is seen by nobody else: its dk, dv are sums over the heads of this row alone.
            static_for<0, 2>([&](auto S) {
                constexpr int s = decltype(S)::value;
                if (!targets[s]) return;
                const int pos = (s == 0 ? OP::ROWS0 : OP::ROWS1) + wave * OP_TILE;
                const PackedRows::Row x = pr.at((NW * s + wave) * 32 + l32);
                const int tok = tok_shift + x.row;
                const bool stores = x.live && tok >= LK && (l32 & (map.heads - 1)) == 0;
                const int64_t koff = ((kv_base + tok) * p.Hkv + g) * D + 8 * hf;
                auto self = [&](auto W) __attribute__((always_inline)) {
#pragma unroll 1
                    for (int ks = 0; ks < NKS; ks++) {
                        const bf16x8 q8 = *(const bf16x8*)at(pos + (nat0 ^ (ks << 5))), do8 = *(const bf16x8*)at(pos + OP::DO + (nat0 ^ (ks << 5)));
                        bf16x8 dk8, dv8;
#pragma unroll
                        for (int j = 0; j < 8; j++) {
                            dk8[j] = (__bf16)sum_lanes<decltype(W)::value>(fk[s] * (float)q8[j]);
                            dv8[j] = (__bf16)sum_lanes<decltype(W)::value>(fv[s] * (float)do8[j]);
                        }
                        if (stores) {
                            *(bf16x8*)((__bf16*)p.dk + koff + ks * 16) = dk8;
                            *(bf16x8*)((__bf16*)p.dv + koff + ks * 16) = dv8;
                        }
                    }
                };
                if (map.heads == 1) self(std::integral_constant<int, 1>{});
                else if (map.heads == 2) self(std::integral_constant<int, 2>{});
                else if (map.heads == 4) self(std::integral_constant<int, 4>{});
                else self(std::integral_constant<int, 8>{});
            });
        }
        __syncthreads();
        // Q^T or dO^T of the first units of the group, features 32 (t % 2) ..: the constant operand of phase 2
        const int rows_t = (t < 2 ? OP::DO : 0) + group * 4 * OP_TILE + (tr0 ^ ((t & 1) << 6));
        bf16x8 ct[4][2];
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) ct[j][s2] = tr64(OP::ROWS0 + rows_t, j * OP_TILE + s2 * 2048);
        __syncthreads();
        const int units[2] = {n_units - 4 * group, n_units - NW - 4 * group};  // of this group: how many first, second ones
        // a unit that does not exist, next to some that do, is there with zero weights
        static_for<0, 2>([&](auto S) {
            constexpr int s = decltype(S)::value;
            if (t >= units[s] && units[s] > 0) {
                const bf16x8 zero = {};
                const int pos = (group * 8 + 4 * s + t) * OP_UNIT + lane * 32;
                *(bf16x8*)at(OP::P + pos) = zero;
                *(bf16x8*)at(OP::P + pos + 16) = zero;
                *(bf16x8*)at(OP::DS + pos) = zero;
                *(bf16x8*)at(OP::DS + pos + 16) = zero;
            }
        });
        wait_vmem_loads();
        lds_barrier();

        // What the groups made of a block's dV^T (t < 2) or dK^T: the other group's sums of this wave's part of the tile added to its
        // own, and the rows of dk, dv stored.
        constexpr int NQ = 4 / NG;  // registers / 4 of the part: with two groups, half of the tile each
        floatx4 mine[NQ];
        auto finish = [&](int i) __attribute__((always_inline)) {
            const int ln = lane_anew();
            if constexpr (NG > 1) {
#pragma unroll
                for (int q = 0; q < NQ; q++) mine[q] += *(const floatx4*)at(OP::X + (wave ^ 4) * 2048 + q * 1024 + ln * 16);
            }
            const float f = PW ? p.scale * p.norm : t < 2 ? 1.f : p.scale;
            const int key = ln & 31;
            static_for<0, NQ / 2>([&](auto H) {
                constexpr int h = decltype(H)::value;
                const bf16x8 o8 = rows_of_16(mine[2 * h], mine[2 * h + 1], f);
                if (32 * i + key < LK) {
                    char* dst = (char*)(t < 2 ? p.dv : p.dk) + 2 * uniform64(((kv_base + 32 * (int64_t)i) * p.Hkv + g) * D + (t & 1) * 32 + group * 16);
                    *(bf16x8*)(dst + 32 * h + (uint32_t)(key * p.Hkv * D * 2 + 16 * (ln >> 5))) = o8;
                }
            });
        };
        // At the start of block i: what block i - 1 still has to do, then block i + 1 is requested, to its stage.
        auto start = [&](int i) __attribute__((always_inline)) {
            if (NG > 1 && i > 0) finish(i - 1);
            if (i + 1 < n_blocks) issue_kv(i + 1);
        };
        // units 0 .. N - 1 of this wave against a block (an, ak: its K/V)
        auto phase1 = [&](auto N, int i, int an, int ak) __attribute__((always_inline)) {
            constexpr int NU = decltype(N)::value;
            const int k0 = 32 * i;
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            const int ar = fresh(OP::ROWS1 + wave * OP_TILE + nat0), aw = fresh((group * 8 + t) * OP_UNIT + pw0());
            floatx16 Sx[NU];  // S^T, as dP^T: [key (registers)][row (lanes)]
            bf16x8 pb[2], dsb[2], kt[NDB][2];
            typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
            auto weights = [&](auto S, const floatx16& dP) __attribute__((always_inline)) {
                constexpr int s = decltype(S)::value;
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    if constexpr (PW) {
                        const float sg = pw_sigmoid(Sx[s][v], neg_c2), pw = pw_silu(Sx[s][v], sg);
                        pb[v / 8][v % 8] = (__bf16)pw;
                        dsb[v / 8][v % 8] = (__bf16)(dP[v] * pw_silu_prime_of(pw, sg, p.scale));
                    } else {
                        const float pw = fast_exp2(fmaf(Sx[s][v], c2, -lse2[s]));
                        pb[v / 8][v % 8] = (__bf16)pw;
                        dsb[v / 8][v % 8] = (__bf16)(pw * (dP[v] + dl[s]));
                    }
                }
            };
            // Register v of the lane holds key 8 (v / 4) + 4 hf + v % 4 of the block.  What a row does not see is cleared
            // bit by bit from the rounded weights, whatever the product with a repeated or real-time key gave.
            // (P and dS in LDS need it only for real-time keys: a key past the end is a column that is not stored.)
            auto clear = [&](auto S, bool own_too, bf16x8 (&x)[2]) __attribute__((always_inline)) {
                constexpr int s = decltype(S)::value;
                const int hf4 = 4 * (lane_anew() >> 5);  // (anew, or the comparisons would be made in every block)
                const int over = hf4 - ((RT ? lim[s] : LK) - k0), mine_k = own[s] - k0 - hf4;
                static_for<0, 8>([&](auto V) {
                    constexpr int v = 2 * decltype(V)::value, key = 8 * (v / 4) + v % 4;
                    const unsigned keep = ((over < -key || (RT && own_too && mine_k == key)) ? 0xffffu : 0u) |
                                          ((over < -key - 1 || (RT && own_too && mine_k == key + 1)) ? 0xffff0000u : 0u);
                    uintx4 d = __builtin_bit_cast(uintx4, x[v / 8]);
                    d[v % 8 / 2] &= keep;
                    x[v / 8] = __builtin_bit_cast(bf16x8, d);
                });
            };
            auto store = [&](auto S) __attribute__((always_inline)) {
                constexpr int s = decltype(S)::value;
                static_for<0, 4>([&](auto Q) {
                    constexpr int q = decltype(Q)::value, o = 4 * (q & 1);
                    *(bf16x4*)at((aw ^ (q << 4)) + OP::P + 4 * s * OP_UNIT) = __builtin_shufflevector(pb[q / 2], pb[q / 2], o, o + 1, o + 2, o + 3);
                    *(bf16x4*)at((aw ^ (q << 4)) + OP::DS + 4 * s * OP_UNIT) = __builtin_shufflevector(dsb[q / 2], dsb[q / 2], o, o + 1, o + 2, o + 3);
                });
            };
            // P and dS of the unit to LDS; then dsb is what dQ adds up (a real-time row's dQ started from its own key)
            auto hand_over = [&](auto S) __attribute__((always_inline)) {
                if constexpr (RT) {
                    if (k0 + 32 > L) clear(S, true, pb), clear(S, true, dsb);
                    store(S);
                    if (k0 + 32 > L) clear(S, false, dsb);
                } else {
                    store(S);
                    if (k0 + 32 > LK) clear(S, false, dsb);
                }
            };
            // dQ^T[d][row] += sum_key K[key][d] dS^T[key][row]
            auto add_dq = [&](auto S) __attribute__((always_inline)) {
                constexpr int s = decltype(S)::value;
#pragma unroll
                for (int db = 0; db < NDB; db++)
#pragma unroll
                    for (int s2 = 0; s2 < 2; s2++) dQ[s][db] = mfma32(kt[db][s2], dsb[s2], dQ[s][db]);
            };
            const std::integral_constant<int, 0> u0{};
            const std::integral_constant<int, NU - 1> u1{};
            // The order of what follows is the point: every read from LDS is issued a step ahead of its use, as many as
            // there are registers for, and the products of one unit have the exponentials of the other behind them.
            auto k_of = [&](int ks) __attribute__((always_inline)) { return *(const bf16x8*)at(an ^ (ks << 5)); };
            auto v_of = [&](int ks) __attribute__((always_inline)) { return *(const bf16x8*)at((an ^ (ks << 5)) + OP_TILE); };
            auto q1_of = [&](int ks) __attribute__((always_inline)) { return *(const bf16x8*)at(ar ^ (ks << 5)); };
            auto do1_of = [&](int ks) __attribute__((always_inline)) { return *(const bf16x8*)at((ar ^ (ks << 5)) + OP::DO); };
            bf16x8 kv[NKS], r1[NKS];
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) {
                kv[ks] = k_of(ks);
                if constexpr (NU > 1) r1[ks] = q1_of(ks);
            }
            start(i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) {
                Sx[0] = mfma32(kv[ks], q0[ks], ks == 0 ? zero : Sx[0]);
                if constexpr (NU > 1) Sx[1] = mfma32(kv[ks], r1[ks], ks == 0 ? zero : Sx[1]);
                kv[ks] = v_of(ks);
            }
            __builtin_amdgcn_sched_barrier(0);
            floatx16 dP;
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) dP = mfma32(kv[ks], do0[ks], ks == 0 ? zero : dP);
            auto fetch_kt = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int db = 0; db < NDB; db++)
#pragma unroll
                    for (int s2 = 0; s2 < 2; s2++) kt[db][s2] = tr64(ak ^ (db << 6), s2 * 2048);
            };
            if constexpr (NU > 1) {
#pragma unroll
                for (int ks = 0; ks < 2; ks++) kv[ks] = v_of(ks), r1[ks] = do1_of(ks);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                fetch_kt();
            }
            weights(u0, dP);
            hand_over(u0);
            if constexpr (NU > 1) {
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    dP = mfma32(kv[ks % 2], r1[ks % 2], ks == 0 ? zero : dP);
                    if (ks + 2 < NKS) kv[ks % 2] = v_of(ks + 2), r1[ks % 2] = do1_of(ks + 2);
                }
                fetch_kt();
            }
            add_dq(u0);
            if constexpr (NU > 1) {
                weights(u1, dP);
                hand_over(u1);
                add_dq(u1);
            }
        };
        const floatx16 zeros = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // ---- the blocks
        for (int i = 0; i < n_blocks; i++) {
            if (ask_late && i + ASK_AHEAD == n_blocks) ask();  // (in front of the block's copies, which are waited for by count)
            const int stage = OP::KV + (i & 1) * OP::STAGE;
            const int an = fresh(stage + nat0), ak = fresh(stage + tr0);
            if (t < units[1]) phase1(std::integral_constant<int, 2>{}, i, an, ak);
            else if (t < units[0]) phase1(std::integral_constant<int, 1>{}, i, an, ak);
            else start(i);
            // dV^T (t < 2) or dK^T of the block, [d (registers)][key (lanes)]: the group's rows
            const int ap = fresh((t < 2 ? OP::P : OP::DS) + group * 8 * OP_UNIT + pr0), at2 = fresh(OP::ROWS1 + rows_t);
            lds_barrier();
            floatx16 acc;
            // step k of 16: rows 16 (k % 2) .. of unit k / 2 of the group.  Reads run AHEAD steps in front of the products.
            constexpr int AHEAD = 4;
            bf16x8 wt[AHEAD], c1[AHEAD];
            auto fetch = [&](auto K) __attribute__((always_inline)) {
                constexpr int k = decltype(K)::value, plus = (k / 2) * OP_UNIT + (k & 1) * 1024;
                wt[k % AHEAD] = lds_read_tr_pair(at(ap + plus), at((ap ^ 32) + plus + 512));
                if constexpr (k >= 8) c1[k % AHEAD] = tr64(at2, (k / 2 - 4) * OP_TILE + (k & 1) * 2048);
            };
            auto steps = [&](auto K) __attribute__((always_inline)) {
                constexpr int n = decltype(K)::value;
                static_for<0, AHEAD>(fetch);
                __builtin_amdgcn_sched_barrier(0);
                static_for<0, n>([&](auto J) {
                    constexpr int k = decltype(J)::value;
                    acc = mfma32(k < 8 ? ct[k % 8 / 2][k & 1] : c1[k % AHEAD], wt[k % AHEAD], k == 0 ? zeros : acc);
                    if constexpr (k + AHEAD < n) fetch(std::integral_constant<int, k + AHEAD>{});
                    if (k & 1) __builtin_amdgcn_sched_barrier(0);
                });
            };
            if (units[1] > 0) steps(std::integral_constant<int, 16>{});
            else if (units[0] > 0) steps(std::integral_constant<int, 8>{});
            else acc = zeros;
            if constexpr (NG > 1) {  // half of the tile to the other group, the other half stays here
                const int x = OP::X + wave * 2048 + lane_anew() * 16;
                if (group == 0) {
                    *(floatx4*)at(x) = __builtin_shufflevector(acc, acc, 8, 9, 10, 11);
                    *(floatx4*)at(x + 1024) = __builtin_shufflevector(acc, acc, 12, 13, 14, 15);
                    mine[0] = __builtin_shufflevector(acc, acc, 0, 1, 2, 3);
                    mine[1] = __builtin_shufflevector(acc, acc, 4, 5, 6, 7);
                } else {
                    *(floatx4*)at(x) = __builtin_shufflevector(acc, acc, 0, 1, 2, 3);
                    *(floatx4*)at(x + 1024) = __builtin_shufflevector(acc, acc, 4, 5, 6, 7);
                    mine[0] = __builtin_shufflevector(acc, acc, 8, 9, 10, 11);
                    mine[1] = __builtin_shufflevector(acc, acc, 12, 13, 14, 15);
                }
            } else {
                static_for<0, NQ>([&](auto Q) {
                    constexpr int q = 4 * decltype(Q)::value;
                    mine[q / 4] = __builtin_shufflevector(acc, acc, q, q + 1, q + 2, q + 3);
                });
                finish(i);
            }
            // block i + 1 of K/V has landed (one group: two stores of this block were issued behind it, in this order)
            if constexpr (NG == 1) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds_barrier();
        }
        if (NG > 1 && n_blocks > 0) finish(n_blocks - 1);
        // ---- dQ
        static_for<0, 2>([&](auto S) {
            constexpr int s = decltype(S)::value;
            const PackedRows::Row x = pr.at((NW * s + wave) * 32 + l32);
            __bf16* op = (__bf16*)p.dq + ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
            static_for<0, NKS>([&](auto Ks) {
                constexpr int ks = decltype(Ks)::value;
                const floatx16& d = dQ[s][ks / 2];
                constexpr int v = 8 * (ks % 2);
                const bf16x8 o8 = rows_of_16(__builtin_shufflevector(d, d, v, v + 1, v + 2, v + 3), __builtin_shufflevector(d, d, v + 4, v + 5, v + 6, v + 7),
                                             PW ? p.scale * p.norm : p.scale);
                if (x.live) *(bf16x8*)(op + 16 * ks) = o8;
            });
        });
    };  // process

    // persistent workgroup: its own index first, then what the work counters give until all lists are exhausted
    for (;;) {
        if (wave == 0) *s_item = queue_resolve(p.queue, xcd, taken, per_xcd, gridDim.x);
        __syncthreads();
        const int id = __builtin_amdgcn_readfirstlane(*s_item);
        if (id < 0) break;
        __syncthreads();  // s_item is free again
        process((unsigned)id);
        __syncthreads();
    }
}

bool power_of_two(int x) { return x > 0 && (x & (x - 1)) == 0; }

// one group per workgroup?
bool single_group(const Params& p) { return max_query_rows(p) * (p.Hq / p.Hkv) <= OnePass<1>::LANES; }

}  // namespace
bool onepass_asks_late(const Params& p) { return mean_keys(p) > 32 * (ASK_AHEAD - 1); }
namespace {

template <int NG, bool RT, bool PW>
hipError_t launch(const Params& p, hipStream_t s) {
    using OP = OnePass<NG>;
    const RowMap map = row_map(OP::LANES, p.Hq, p.Hkv, max_query_rows(p));
    const int64_t n_items = work_grid((int64_t)p.batch * p.Hkv, 1);
    if (n_items >= (1ll << 31)) return hipErrorInvalidValue;
    const int64_t resident = resident_workgroups<bwd_onepass_kernel<NG, RT, PW>>(OP::NW * 64);
    Params pk = p;
    pk.queue = p.queue + QUEUE_DKDV * N_XCD;
    hipLaunchKernelGGL((bwd_onepass_kernel<NG, RT, PW>), dim3((unsigned)std::min(n_items, resident)), dim3(OP::NW * 64), 0, s, pk, map,
                       (unsigned)(n_items / N_XCD), onepass_asks_late(p));
    return hipGetLastError();
}
template <int NG>
hipError_t launch(const Params& p, hipStream_t s) {
    if (p.pointwise) return p.rt_len ? launch<NG, true, true>(p, s) : launch<NG, false, true>(p, s);
    return p.rt_len ? launch<NG, true, false>(p, s) : launch<NG, false, false>(p, s);
}

}  // namespace

// Which calls: those whose users' pairs fit, and whose estimated time is below that of the other forms by a margin that covers what
// the estimates miss.  Both (us): two passes cost by items (users x kv heads) x units x blocks of 32 keys, by the rows and the keys they read,
// and by the longest user; here an item costs a prologue and its blocks, 512 (256) of them run at a time and the last round takes as long as
// any.  The longest item counts with the most pairs that a user has, not with the mean's: 160 users of up to 3407 keys x 75
// candidates, 8/2 heads, take 234 us in two passes and 293 here.  Three fits, since what the passes are made of changes: full layers; target
// layers on less than 512 keys; and on more, where two passes may keep a user's rows resident.
// The fits are of 7808 calls timed in both forms (full and target layers; 1..512 pairs, 16..4145 keys, 76..15952 items; with real-time tokens
// and pointwise weights, too), both of which took their next items early then and stored results in narrower words.  As the kernels are, 2400 calls of
// all forms, 334 of which fit one pass and are not brief: one pass takes 0.88 of the time of two and is faster on 243.  Where it is not, a few workgroups
// make a second round (there it has to win by a fifth) or most units are idle.  The line takes 195, at 0.81 of the time, eight of them slower than in two
// passes by more than 3 %; of the 139 that it leaves 57 would be faster by more than that, which is 7 % of the time of the 139.
static bool onepass_fits(const Params& p) {
    const int r = p.Hq / p.Hkv;
    return p.d == OP_D && power_of_two(r) && r <= OP_MAX_HEADS && p.total_q > 0 && max_query_rows(p) * r <= OnePass<2>::LANES;
}
// target layers on long histories, whose two passes may keep a user's rows resident
static bool long_histories(const Params& p) { return p.layer != 0 && mean_keys(p) >= 512.; }
static double onepass_rounds(const Params& p) { return (double)p.batch * p.Hkv * (single_group(p) ? 1 : 2) / 512.; }

double onepass_us(const Params& p) {
    if (!onepass_fits(p)) return INFINITY;
    const double r = p.Hq / p.Hkv, pairs = mean_rows(p) * r, most = max_query_rows(p) * r, keys = mean_keys(p), longest = (double)max_lead_keys(p);
    const int groups = single_group(p) ? 1 : 2;
    const double rounds = onepass_rounds(p), whole = std::ceil(rounds - 0.01);
    struct { double launch, fixed, unit, block, second, alone, alone_second, partial, jagged, rt, pw; } c;
    if (long_histories(p)) c = groups == 2     ? decltype(c){16.6, 7.7, 0.6, 1.85, 0.5, 1.85, 0.5, 0., 0.55, 1.1, 1.035}
                               : rounds <= 0.5 ? decltype(c){5.6, 17.9, 1.2, 1.5, 0.69, 1.16, 0.35, 0., 0.55, 1.1, 1.035}
                                               : decltype(c){16.6, 17.9, 1.2, 1.5, 0.69, 1.16, 0.35, 0., 0.55, 1.1, 1.035};
    else if (groups == 1) c = {5.6, 7.6, 0.96, 1.8, 0.72, 1.2, 0.34, 0.39, 0.44, 1.1, 0.99};
    else c = {5.1, 5.9, 0.65, 2.1, 0.47, 1.1, 1.3, 0.18, 0.48, 1.1, 0.93};
    const double first_units = 128. * groups;  // pairs that the waves hold with one unit each
    auto two_units = [&](double x) { return most > first_units ? std::min(1., std::max(0., (x - first_units) / (0.25 * first_units) + 0.5)) : 0.; };
    const double fixed = c.fixed + c.unit * (pairs / 32. + 0.5);
    const double item = fixed + (c.block + c.second * two_units(pairs)) * (keys / 32. + 0.5);
    const double last = fixed + (c.alone + c.alone_second * two_units(most)) * longest / 32.;  // of the longest item
    const double many = keys >= 0.9 * longest ? whole + c.partial * (rounds - whole) : std::max(rounds + c.jagged, 1.);
    return c.launch + std::max(last, many * item) * (p.rt_len ? c.rt : 1.) * (p.pointwise ? c.pw : 1.);
}

bool bwd_is_onepass(const Params& p) {
    if (!onepass_fits(p) || bwd_is_brief(p)) return false;
    const double items = (double)p.batch * p.Hkv, r = p.Hq / p.Hkv, units = mean_rows(p) * r / 32. + 0.5, blocks = mean_keys(p) / 32. + 0.5;
    const bool resident = long_histories(p);
    struct { double launch, product, pw, rt, unit, block, item, longest, most, rt_launch; } t;
    if (p.layer == 0) t = {5.7, 0.36, 0.95, 2.5, 6.0, 7.1, 6.4, 0.26, 0.36, 1.0};
    else if (resident) t = {10.4, 0.67, 1.4, 1.43, 9.4, 4.6, 0., 0.34, 0.2, 0.};
    else t = {3.9, 0.62, 1.4, 1.2, 8.1, 4.6, 5.1, 0.32, 0.67, 2.8};
    const double product = t.product * (p.pointwise ? t.pw : 1.) * (p.rt_len ? t.rt : 1.);
    const double two_passes = t.launch + (p.rt_len ? t.rt_launch : 0.) + (t.longest * max_lead_keys(p) + t.most * max_query_rows(p) * r) / 32. +
                              items / 1024. * (product * units * blocks + t.unit * units + t.block * blocks + t.item);
    const double one_pass = onepass_us(p), rounds = onepass_rounds(p);
    return resident ? one_pass + 5. < two_passes : one_pass < two_passes * (rounds > 1.02 && rounds < 1.5 ? 0.8 : 0.93);
}

hipError_t launch_bwd_onepass_bf16(const Params& p, hipStream_t s) {
    timing_begin(MTFM_HTA_KERNEL_BWD_DKDV, s);
    const hipError_t e = single_group(p) ? launch<1>(p, s) : launch<2>(p, s);
    timing_end(MTFM_HTA_KERNEL_BWD_DKDV, s);
    return e;
}

}  // namespace hta
