// bf16 backward of Hybrid Target Attention for calls of little work (gfx950): a few dozen users, short histories or few
// candidates.  Same mask, products and results as the two passes of hta_bwd_bf16.hip; what differs is the shape.  There,
// a wave walks all keys of its rows (or all rows of its keys) alone, which on a call that fills the chip for a few
// microseconds only makes a long chain: 19 users of 1000 keys x 40 candidates spent 49 us in the dQ and 56 us in the dK/dV pass
// on 2 us of matrix work.
//
// Two launches:
//   1. prepare: -delta = -<dO, O> and -lse/scale of every row (and the rows' limits, with real-time tokens), for
//   2. one grid of three kinds of workgroups that do not depend on each other:
//      dK/dV: 32 keys; the four waves share the rows, every fourth unit of 32 packed (row, head) pairs each, and add up
//             their dK, dV through LDS.  Or 128 keys, 32 to a wave, each with all units to itself: where users have few rows four waves
//             have nothing to share, and a workgroup costs 4 to 6 us beside its units (whole backward of 277 target layers of 1..4 candidates
//             on 241 keys, 8/2 heads, 57 -> 31 us; 40 of 1..4 on 881..1762, 16/2 heads at head_dim 128, 113 -> 48);
//      dQ:    32 packed rows; the four waves share the keys, every fourth block of 32 each, and add up their dQ;
//      dk/dv of the target tokens' own keys.
// A wave only reads what it copied itself (global -> LDS, asynchronously, two units or blocks ahead): no barrier before
// the final sums.  Sums are formed in a fixed order: the results are bitwise reproducible.
#include "../../include/mtfm_hta.h"
#include "../../include/mtfm_hta_timing.h"
#include "hta_bwd_self.h"
#include "hta_common.h"
#include "hta_dkdv_brief.h"
#include "hta_mfma.h"
#include "hta_rows.h"
#include "hta_tiles.h"

#include <algorithm>
#include <cmath>

namespace hta {
namespace {

constexpr int NW = BRIEF_NW;

// What the one grid can look like.  Four waves per key block or one, and with one the dQ workgroups, whose chains are then no shorter, in
// front or behind.
// (Two waves per block, which are never far behind the better of these, 0.3 % of the time; dQ in front with four, 0.2 %: not worth their kernels.)
struct BriefForm {
    int ways;
    bool dq_first;
    double us;  // estimated
};
// Time of a call in that form (us): what the workgroups take together -- a fixed part, a part per step (a unit of rows; four blocks of keys),
// and what one costs that only the longest user has a tile for -- or the longest chain, whichever is longer (the cubes: near the line a bit of
// both).  Fits of 13000 calls timed in every form (4 to 600 users of 32 to 4096 keys, 2 to 160 candidates, full and target layers):
// of 6370 short calls the form with the least takes 0.74 of the time of four waves per block, the best of each 0.73; 2 % are slower by more than 3 %.
double brief_us(const Params& p, int ways, bool dq_first, double chain_keys) {
    struct { double launch, kv, kv_step, dq, dq_step, empty, chain, chain_kv, chain_dq, rt, pw; } c;
    if (p.d == 32) c = ways == 4 ? decltype(c){6.7, 1.7, 0.55, 0.9, 1.2, 0.7, 0.96, 0.59, 0.46, 1.37, 1.18}
                     : !dq_first ? decltype(c){6.2, 4.2, 0.76, 0.6, 0.72, 1.1, 1.3, 0.6, 0.37, 1.55, 1.29}
                                 : decltype(c){6.1, 3.0, 1.44, 1.7, 0.3, 0.63, 1.4, 0.65, 0.33, 1.54, 1.29};
    else if (p.d == 64) c = ways == 4 ? decltype(c){7.4, 4.3, 0.4, 3.7, 2.1, 1.2, 0., 1.03, 0.98, 1.15, 1.09}
                          : !dq_first ? decltype(c){7.1, 6.9, 0.81, 3.1, 1.5, 2.2, 0.94, 0.84, 0.63, 1.41, 1.16}
                                      : decltype(c){7.3, 5.4, 2.25, 4.85, 0.32, 1.9, 0.63, 0.96, 0.54, 1.39, 1.15};
    else c = ways == 4 ? decltype(c){8.0, 5.9, 0.8, 5.85, 2.55, 1.8, 0., 1.39, 1.96, 1.05, 1.1}
           : !dq_first ? decltype(c){7.4, 9.8, 2.4, 5.2, 0.44, 3.4, 2.55, 1.2, 1.1, 1.19, 1.14}
                       : decltype(c){8.1, 8.5, 2.64, 6.8, 0.3, 2.7, 1.4, 1.53, 0.89, 1.19, 1.13};
    const double groups = (double)p.batch * p.Hkv, r = p.Hq / p.Hkv, keys = mean_keys(p), longest = (double)max_lead_keys(p);
    const double units = mean_rows(p) * r / 32., most = (double)max_query_rows(p) * r / 32., block = NW / ways * 32.;
    const double kv_grid = groups * std::ceil(longest / block), kv = std::min(groups * (keys / block + 0.5), kv_grid);
    const double dq_grid = groups * std::ceil(most), dq = std::min(groups * (units + 0.5), dq_grid);
    const double step = (p.rt_len ? c.rt : 1.) * (p.pointwise ? c.pw : 1.);
    const double all = (c.kv * kv + c.dq * dq + c.empty * (kv_grid - kv + dq_grid - dq) +
                        step * (c.kv_step * kv * std::max(1., units / ways + 0.25) + c.dq_step * dq * std::max(1., keys / 128. + 0.3))) / (p.d == 128 ? 256. : 512.);
    const double chain = c.chain + step * std::max(c.chain_kv * std::ceil(most / ways), c.chain_dq * std::ceil(chain_keys / 128.));
    return c.launch + std::cbrt(all * all * all + chain * chain * chain);
}
// The form with the least time, but four waves while the workgroups with work take less than a fifth of the chip: nothing waits there, and the
// chain of a block that four waves share is the shorter one, which the estimates do not tell within a microsecond.  The chains are those of the
// mean user, since the bounds may be far above all lengths.  (1223 target layers with true bounds and 2260 with bounds of 1.5 to 8 times the
// longest: 2 % of both are slower than with four waves by more than 3 %, where the estimates with the longest user by the bounds alone had 9 and
// 15 %; times the best form's: 1.008 and 1.015, before 1.011 and 1.029.)
BriefForm brief_form(const Params& p) {
    const double groups = (double)p.batch * p.Hkv, slots = p.d == 128 ? 256. : 512.;
    const double work = groups * (mean_keys(p) / 32. + 0.5) + groups * (mean_rows(p) * (p.Hq / p.Hkv) / 32. + 0.5);
    BriefForm best = {4, false, brief_us(p, 4, false, mean_keys(p))};
    if (work > 0.2 * slots)
        for (bool dq_first : {false, true}) {
            const double us = brief_us(p, 1, dq_first, mean_keys(p));
            if (us < best.us) best = {1, dq_first, us};
        }
    best.us = brief_us(p, best.ways, best.dq_first, (double)max_lead_keys(p));
    return best;
}
// The same for the two passes (in whichever of their forms): dQ by tiles of 128 packed rows, dK/dV by 128 keys.
double two_passes_us(const Params& p) {
    struct { double launch, dq, dq_step, kv, kv_step, chain, chain_dq, chain_kv, rt, pw; } c;
    if (p.d == 32) c = {10.6, 2.9, 1.55, 3.4, 0.73, 0., 0.83, 0.17, 1.33, 1.35};
    else if (p.d == 64) c = {11.6, 4.6, 1.13, 6.4, 1.9, 0.9, 1.39, 0.25, 1.22, 1.24};
    else c = {17.2, 18.1, 8.3, 13.7, 1.6, 0.3, 2.3, 0.36, 1.14, 1.17};
    const double groups = (double)p.batch * p.Hkv, r = p.Hq / p.Hkv, keys = mean_keys(p), units = mean_rows(p) * r / 32.;
    const double dq = groups * (units / 4. + 0.5), kv = groups * (keys / 128. + 0.5), step = (p.rt_len ? c.rt : 1.) * (p.pointwise ? c.pw : 1.);
    const double all = (c.dq * dq + c.kv * kv + step * (c.dq_step * dq * keys / 64. + c.kv_step * kv * std::max(1., units))) / 512.;
    const double chain = c.chain + step * (c.chain_dq * max_lead_keys(p) / 64. + c.chain_kv * max_query_rows(p) * r / 32.);
    return c.launch + std::cbrt(all * all * all + chain * chain * chain);
}

// ---------------------------------------------------------------------------------------- dQ
template <int D, bool RT, bool PW>
__device__ __forceinline__ void brief_dq(const Params& p, const RowMap& map, unsigned id, unsigned char* smem) {
    using BR = Brief<D, RT>;
    constexpr int NKS = D / 16, NDB = D / 32, CPT = BR::CPT;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const int ny = p.Hkv * map.n_chunks;
    const WorkItem w = decode_work(id, p.batch * ny, ny, map.n_tiles);
    if (!w.valid) return;
    const int b = w.user_slot;
    const int g = map.n_chunks == 1 ? w.y : w.y / map.n_chunks, chunk = w.y - g * map.n_chunks;
    const int L = p.hist_len[b], T = p.n_targets[b];
    const int64_t q_base = p.q_off[b], kv_base = p.kv_off[b];
    const int LK = L + (RT ? p.rt_len[b] : 0);
    const int n_rows = p.layer == 0 ? LK + T : T, tok_shift = p.layer == 0 ? 0 : LK;
    if (w.tile * map.rows >= n_rows) return;  // uniform for the workgroup
    const PackedRows pr(map, w.tile, chunk, n_rows, g, p.Hq / p.Hkv);
    const float c2 = p.scale * LOG2E;
    const int n_kb = (LK + 31) / 32, n_mine = n_kb > wave ? (n_kb - wave + NW - 1) / NW : 0;

    uint32_t voff[CPT];
#pragma unroll
    for (int j = 0; j < CPT; j++) {
        const int trow = j * BR::RPC + lane / BR::CPR;
        voff[j] = (uint32_t)((trow * p.Hkv * D + (((lane % BR::CPR) ^ swizzle<D>(trow)) << 3)) * 2);
    }
    const uint32_t lds0 = lds_address(smem) + (uint32_t)wave * BR::SLOTS * BR::KV_BYTES;
    const __bf16* kg = (const __bf16*)p.k + (int64_t)g * D;
    const __bf16* vg = (const __bf16*)p.v + (int64_t)g * D;
    auto issue = [&](int i) __attribute__((always_inline)) {
        if (i >= n_mine) return;
        const int k0 = (wave + i * NW) * 32;
        const int64_t base = (kv_base + k0) * p.Hkv * D;
        const uint32_t dst = lds0 + (uint32_t)(i & 1) * BR::KV_BYTES;
        const bool whole = k0 + 32 <= LK;
#pragma unroll
        for (int j = 0; j < CPT; j++) {
            uint32_t off = voff[j];
            if (!whole) off -= (uint32_t)max(j * BR::RPC + lane / BR::CPR - (LK - 1 - k0), 0) * (uint32_t)(p.Hkv * D * 2);
            copy16_global_to_lds_at(kg + base, off, dst + j * 1024);
            copy16_global_to_lds_at(vg + base, off, dst + BR::TILE * 2 + j * 1024);
        }
    };
    issue(0);
    issue(1);

    int nat[NKS], tlo[NDB], thi[NDB];
    natural_offsets<D>(nat, lane);
    transposed_offsets<D>(tlo, thi, lane);
    const PackedRows::Row x = pr.at(l32);
    bf16x8 qf[NKS], dof[NKS];
    {
        const int64_t off = ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            qf[ks] = *(const bf16x8*)((const __bf16*)p.q + off + ks * 16);
            dof[ks] = *(const bf16x8*)((const __bf16*)p.dout + off + ks * 16);
        }
    }
    const int64_t stat = (int64_t)x.h * p.total_q + q_base + x.row;
    const float lse2 = PW ? 0.f : p.lse[stat] * LOG2E, dl = PW ? 0.f : p.neg_delta[stat];
    const int lim = RT ? p.lim[q_base + x.row] : L;
    floatx16 dQ[NDB];  // dQ^T: [d (registers)][row (lanes)]
#pragma unroll
    for (int db = 0; db < NDB; db++)
#pragma unroll
        for (int v = 0; v < 16; v++) dQ[db][v] = 0.f;
    if (wave == 0 && tok_shift + x.row >= L) {  // own key of target and real-time rows
        const int64_t off = ((kv_base + tok_shift + x.row) * p.Hkv + g) * D;
        bf16x8 kk[NKS], vv[NKS];
        bf16x4 kt[NDB][4];
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            kk[ks] = *(const bf16x8*)((const __bf16*)p.k + off + ks * 16 + 8 * hf);
            vv[ks] = *(const bf16x8*)((const __bf16*)p.v + off + ks * 16 + 8 * hf);
        }
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int v4 = 0; v4 < 4; v4++) kt[db][v4] = *(const bf16x4*)((const __bf16*)p.k + off + db * 32 + 8 * v4 + 4 * hf);
        float sp = 0.f, dpp = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            sp = dot_bf16x8(sp, qf[ks], kk[ks]);
            dpp = dot_bf16x8(dpp, dof[ks], vv[ks]);
        }
        sp += other_half(sp);
        dpp += other_half(dpp);
        float ds;
        if constexpr (PW) ds = dpp * pw_silu_prime(sp * p.scale, pw_sigmoid(sp, -c2));
        else ds = fast_exp2(fmaf(sp, c2, -lse2)) * (dpp + dl);
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int v4 = 0; v4 < 4; v4++)
#pragma unroll
                for (int j = 0; j < 4; j++) dQ[db][4 * v4 + j] = ds * (float)kt[db][v4][j];
    }
    wait_vmem_loads();

    auto block = [&](int i, auto Tail) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(Tail)::value;
        if (i + 1 < n_mine) wait_vmem_outstanding<2 * CPT>(); else wait_vmem_outstanding<0>();
        const int k0 = (wave + i * NW) * 32;
        const __bf16* Ks = (const __bf16*)(smem + (wave * BR::SLOTS + (i & 1)) * BR::KV_BYTES);
        const __bf16* Vs = Ks + BR::TILE;
        floatx16 S, dP;  // S^T, dP^T: [key (registers)][row (lanes)]
#pragma unroll
        for (int v = 0; v < 16; v++) S[v] = 0.f, dP[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            S = mfma32(*(const bf16x8*)(Ks + nat[ks]), qf[ks], S);
            dP = mfma32(*(const bf16x8*)(Vs + nat[ks]), dof[ks], dP);
        }
        bf16x8 kt[NDB][2];
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) kt[db][s2] = lds_read_tr_pair(Ks + 16 * s2 * D + tlo[db], Ks + 16 * s2 * D + thi[db]);
        // keys past the row's limit are not visible (P = 0)
        const int over = 4 * hf - (min(lim, LK) - k0);
        bf16x8 dsb[2];
        static_for<0, 16>([&](auto V) {
            constexpr int v = decltype(V)::value;
            if constexpr (TAIL) S[v] = over >= -(8 * (v / 4) + (v % 4)) ? (PW ? PW_MASKED : -INFINITY) : S[v];
            if constexpr (PW) {
                dsb[v / 8][v % 8] = (__bf16)(dP[v] * pw_silu_prime_of_logit(S[v], pw_sigmoid(S[v], -c2), p.scale));
            } else {
                dsb[v / 8][v % 8] = (__bf16)(fast_exp2(fmaf(S[v], c2, -lse2)) * (dP[v] + dl));
            }
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(i + 2);
        // dQ^T[d][row] += sum_key K[key][d] dS^T[key][row]
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) dQ[db] = mfma32(kt[db][s2], dsb[s2], dQ[db]);
    };
    const int n_whole = min(max(L / 32 - wave + NW - 1, 0) / NW, n_mine);
    for (int i = 0; i < n_whole; i++) block(i, std::false_type{});
    for (int i = n_whole; i < n_mine; i++) block(i, std::true_type{});

    lds_barrier();
    float* acc = (float*)smem;  // [wave][row][ROW_PITCH]
    {
        float* o = acc + (wave * 32 + l32) * BR::ROW_PITCH + 4 * hf;
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int v4 = 0; v4 < 4; v4++) {
                floatx4 y;
#pragma unroll
                for (int j = 0; j < 4; j++) y[j] = dQ[db][4 * v4 + j];
                *(floatx4*)(o + db * 32 + 8 * v4) = y;
            }
    }
    lds_barrier();
    constexpr int QUADS = D / 4;
    const float f = PW ? p.scale * p.norm : p.scale;
    for (int e = tid; e < 32 * QUADS; e += NW * 64) {
        const int c = e % QUADS, l = e / QUADS;
        const PackedRows::Row y = pr.at(l);
        if (!y.live) continue;
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NW; k++) o += *(const floatx4*)(acc + (k * 32 + l) * BR::ROW_PITCH + 4 * c);
        bf16x4 o4;
#pragma unroll
        for (int j = 0; j < 4; j++) o4[j] = (__bf16)(o[j] * f);
        *(bf16x4*)((__bf16*)p.dq + ((q_base + y.row) * p.Hq + y.h) * D + 4 * c) = o4;
    }
}

// n_kv blocks of dK/dV and n_dq of dQ, one kind after the other; then the own keys of the targets, self_bpu blocks per user.
template <int D, int WAYS, bool RT, bool PW>
__global__ __launch_bounds__(NW * 64, D == 128 ? 1 : 2) void brief_kernel(Params p, RowMap map, int n_kt, unsigned n_kv, unsigned n_dq, bool dq_first,
                                                                          unsigned self_bpu) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[Brief<D, RT>::BYTES];
    const unsigned id = blockIdx.x, kv0 = dq_first ? n_dq : 0, dq0 = dq_first ? 0 : n_kv;
    if (id - kv0 < n_kv) brief_dkdv<D, WAYS, RT, PW>(p, map, id - kv0, n_kt, 0, smem);
    else if (id - dq0 < n_dq) brief_dq<D, RT, PW>(p, map, id - dq0, smem);
    else bwd_self_block<D, PW, NW * 64>(p, (int)((id - n_kv - n_dq) % self_bpu), (int)((id - n_kv - n_dq) / self_bpu));
}

// the dK/dV part alone, behind the ordinary dQ pass
template <int D, int WAYS, bool RT, bool PW>
__global__ __launch_bounds__(NW * 64, D == 128 ? 1 : 2) void brief_dkdv_kernel(Params p, RowMap map, int n_kt, int spread) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[Brief<D, RT>::BYTES];
    brief_dkdv<D, WAYS, RT, PW>(p, map, blockIdx.x, n_kt, spread, smem);
}

// -delta and -lse/scale of every (row, head): D/8 lanes each, 16 bytes per lane, rows and heads as they lie in memory.
// (Pointwise weights have neither: zeros, which leaves rows that do not exist to the sentinel.)  Blocks n_stat ..: the
// rows' limits of mask rule 2, lim_bpu blocks per user.
template <int D, bool PW>
__global__ __launch_bounds__(256) void prepare_kernel(Params p, unsigned n_stat, unsigned lim_bpu) {
    if (blockIdx.x >= n_stat) {
        const unsigned id = blockIdx.x - n_stat;
        rt_limit_of_row(p, (int)(id / lim_bpu), (int)(id % lim_bpu) * 256 + threadIdx.x);
        return;
    }
    constexpr int LPR = D / 8;
    const int64_t item = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    const int sub = threadIdx.x % LPR;
    if (item == 0 && sub == 0) p.neg_lse_s[(int64_t)p.Hq * p.total_q] = -1e30f;
    if (item >= p.total_q * p.Hq) return;
    const int64_t row = item / p.Hq, stat = (item - row * p.Hq) * p.total_q + row;
    float delta = 0.f, lse = 0.f;
    if constexpr (!PW) {
        const bf16x8 d8 = *(const bf16x8*)((const __bf16*)p.dout + item * D + 8 * sub);
        const bf16x8 o8 = *(const bf16x8*)((const __bf16*)p.out + item * D + 8 * sub);
        lse = p.lse[stat];
        delta = group_sum(dot_bf16x8(0.f, d8, o8), LPR);
    }
    if (sub == 0) {
        p.neg_delta[stat] = -delta;
        p.neg_lse_s[stat] = -lse / p.scale;
    }
}

template <int D, int WAYS, bool PW>
hipError_t launch(const Params& p, const BriefForm& form, hipStream_t s) {
    const int64_t rows = max_query_rows(p), keys = max_lead_keys(p);
    constexpr int LPR = D / 8, IPB = NW * 64 / LPR;
    const int64_t n_stat = (p.total_q * p.Hq + 256 / LPR - 1) / (256 / LPR);
    const int64_t lim_bpu = p.rt_len ? (rows + 255) / 256 : 0;
    const RowMap map = row_map(32, p.Hq, p.Hkv, rows);
    constexpr int KEYS = NW / WAYS * 32;
    const int64_t n_kt = (keys + KEYS - 1) / KEYS;
    const int64_t n_kv = work_grid((int64_t)p.batch * p.Hkv, n_kt);
    const int64_t n_dq = work_grid((int64_t)p.batch * p.Hkv * map.n_chunks, map.n_tiles);
    const int64_t self_bpu = ((int64_t)p.max_targets * p.Hkv + IPB - 1) / IPB;
    const int64_t n_blocks = n_kv + n_dq + self_bpu * p.batch;
    if (n_stat + lim_bpu * p.batch >= (1ll << 31) || n_blocks >= (1ll << 31)) return hipErrorInvalidValue;
    timing_begin(MTFM_HTA_KERNEL_BWD_DQ, s);
    if (n_stat > 0)
        hipLaunchKernelGGL((prepare_kernel<D, PW>), dim3((unsigned)(n_stat + lim_bpu * p.batch)), dim3(256), 0, s, p,
                           (unsigned)n_stat, (unsigned)(lim_bpu > 0 ? lim_bpu : 1));
    timing_end(MTFM_HTA_KERNEL_BWD_DQ, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    timing_begin(MTFM_HTA_KERNEL_BWD_DKDV, s);
    auto kernel = p.rt_len ? brief_kernel<D, WAYS, true, PW> : brief_kernel<D, WAYS, false, PW>;
    if (n_blocks > 0)
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_blocks), dim3(NW * 64), 0, s, p, map, (int)n_kt, (unsigned)n_kv, (unsigned)n_dq,
                           form.dq_first, (unsigned)(self_bpu > 0 ? self_bpu : 1));
    timing_end(MTFM_HTA_KERNEL_BWD_DKDV, s);
    return hipGetLastError();
}

template <int D, bool PW>
hipError_t launch_form(const Params& p, hipStream_t s) {
    const BriefForm form = brief_form(p);
    return form.ways == 4 ? launch<D, 4, PW>(p, form, s) : launch<D, 1, PW>(p, form, s);
}

template <int D, int WAYS, bool PW>
hipError_t launch_dkdv(const Params& p, hipStream_t s) {
    const int64_t keys = max_lead_keys(p);
    const RowMap map = row_map(32, p.Hq, p.Hkv, max_query_rows(p));
    constexpr int KEYS = NW / WAYS * 32;
    const int64_t n_kt = (keys + KEYS - 1) / KEYS, groups = (int64_t)p.batch * p.Hkv;
    const int spread = grid_spread(p, groups, n_kt);
    const int64_t n_blocks = work_grid(groups, n_kt, spread);
    if (n_blocks >= (1ll << 31)) return hipErrorInvalidValue;
    auto kernel = p.rt_len ? brief_dkdv_kernel<D, WAYS, true, PW> : brief_dkdv_kernel<D, WAYS, false, PW>;
    if (n_blocks > 0) hipLaunchKernelGGL(kernel, dim3((unsigned)n_blocks), dim3(NW * 64), 0, s, p, map, (int)n_kt, spread);
    return hipGetLastError();
}

template <int D, bool PW>
hipError_t launch_dkdv_ways(const Params& p, hipStream_t s) {
    const int ways = dkdv_brief_ways(p);
    return ways == 4 ? launch_dkdv<D, 4, PW>(p, s) : ways == 2 ? launch_dkdv<D, 2, PW>(p, s) : launch_dkdv<D, 1, PW>(p, s);
}

}  // namespace

// Both launches pay where the dQ part is small too: its workgroups of 32 rows walk their keys in a quarter of the time, at
// twice the traffic (19 users of 405..1623 keys x 40 candidates: 66 -> 41 us per step against the ordinary dQ pass and this
// dK/dV pass; 53 users of 100 keys, full layer: 54 either way).  Up to the first line always, beyond it by the estimates, where key
// blocks are not shared.  The lines are fits of 9355 calls, made when the other forms took their next items early and stored results in narrower words.  As
// the kernels are, of 2400 calls 1622 go here, at 0.65 of the time of the better of one pass and two (32, 64 and 128 features alike); 90 of them are slower by
// more than 3 %, 28 of the 227 at head_dim 128; of the others 87 would be faster here by more than that, which is 1.5 % of their time.  The estimate
// of one pass is above its time by a seventh in this range, and further for a row or two on long histories.
bool bwd_is_brief(const Params& p) {
    if (p.total_q == 0) return false;
    const int r = p.Hq / p.Hkv;
    const double blocks = p.total_q * r / 32. * p.Hkv + 0.5 * p.batch * p.Hkv;  // of 32 packed rows
    if (blocks <= 1024. && blocks * (mean_keys(p) / 32. + 0.5) <= 12. * 1024.) return true;
    if (blocks > 4096. || blocks * (mean_keys(p) / 32. + 0.5) > 144. * 1024.) return false;
    const BriefForm form = brief_form(p);
    return form.ways == 1 && form.us < 0.95 * two_passes_us(p) && form.us < 0.8 * onepass_us(p);
}

int bwd_brief_ways(const Params& p, bool* dq_first) {
    const BriefForm form = brief_form(p);
    *dq_first = form.dq_first;
    return form.ways;
}

hipError_t launch_bwd_brief_bf16(const Params& p, hipStream_t s) {
    switch (p.d) {
        case 32: return p.pointwise ? launch_form<32, true>(p, s) : launch_form<32, false>(p, s);
        case 64: return p.pointwise ? launch_form<64, true>(p, s) : launch_form<64, false>(p, s);
        default: return p.pointwise ? launch_form<128, true>(p, s) : launch_form<128, false>(p, s);
    }
}

// Which dK/dV pass takes a call: 0, the ordinary one (or, within it, the one with a user's rows resident in LDS), or the number
// of waves that share a key block's rows here.  From fits of measured times (us): a workgroup costs `fixed` plus `unit`
// per 32-row unit of a wave, the chip holds `slots` of them, and the longest one bounds the call from below.  The ordinary
// pass shares its staging among 128 keys and wins in the long run; it loses where a user's rows walked one after the
// other take longer than the rest of the call.  (The fits are of kernels that took their next items early and stored results in narrower words.  As
// the kernels are, whole backward passes of 583 calls in two passes: the 520 that share rows 0.84 of the ordinary pass's time, the choice 1.024 of
// the best one's.  8/2 heads, ordinary against the best that shares: 64 users of 128..512 keys 91 and 95 us, 19 of 374..1498 209 and 195, 256 of 512..1024
// 1287 and 1474; 16/4 heads, resident against that: 512 x 128 candidates on 512..2048 keys 1.40 ms and 1.79, 64 x 8..32 on 512 keys 41.6 us and 40.5.)
int dkdv_brief_ways(const Params& p) {
    if (p.total_q == 0) return 0;
    const int r = p.Hq / p.Hkv;
    const bool wide = p.d == 128;
    const double slots = wide ? 256. : 512., groups = (double)p.batch * p.Hkv, keys = mean_keys(p);
    const double rows = mean_rows(p), most = (double)max_query_rows(p);
    const double jag = 1. + 0.3 * (most / std::max(rows, 1.) - 1.);  // of rows x keys, over the product of their means
    auto estimate = [&](double workgroups, double mean, double longest) {
        return std::max(workgroups / slots * mean * jag + 0.5 * mean, longest);
    };
    // (the ordinary pass takes 32 rows of one head at a time)
    const double fixed = wide ? 6. : 5.3, unit = (wide ? 1.1 : 1.05) * r;
    // (the resident one walks all keys of a user, past all row blocks that the longest one has, 256 users' kv heads at a time)
    const double blocks = std::min(rows / 32. + 0.5, std::ceil(most / 32.)), users = groups / 256.;
    const double rounds = keys >= 0.9 * (double)max_lead_keys(p) ? std::ceil(users) : std::max(1., users);
    double best = dkdv_is_resident(p)
                      ? 30. + rounds * (keys / 32. + 2.) * (r * blocks + 2.2) * 0.118
                      : estimate(groups * (keys / 128. + 0.5), fixed + unit * (rows / 32. + 0.5), 0.95 * (fixed + unit * (most / 32. + 0.5)));
    int ways = 0;
    for (int w = 1; w <= NW; w *= 2) {
        const double f = wide ? 4. : 3.6, u = wide ? 1.7 : 1.23;
        const double us = estimate(groups * (keys / (128. / w) + 0.5), f + u * std::max(1., rows * r / 32. / w + 0.25),
                                   f + u * (most * r / 32. / w + 0.5));
        if (us < best) best = us, ways = w;
    }
    return ways;
}

hipError_t launch_dkdv_brief_bf16(const Params& p, hipStream_t s) {
    switch (p.d) {
        case 32: return p.pointwise ? launch_dkdv_ways<32, true>(p, s) : launch_dkdv_ways<32, false>(p, s);
        case 64: return p.pointwise ? launch_dkdv_ways<64, true>(p, s) : launch_dkdv_ways<64, false>(p, s);
        default: return p.pointwise ? launch_dkdv_ways<128, true>(p, s) : launch_dkdv_ways<128, false>(p, s);
    }
}

}  // namespace hta
