// The dK/dV pass of 32 keys per workgroup, its four waves sharing the rows (see hta_bwd_brief_bf16.hip for calls of little
// work; the keys behind the history, in calls with real-time tokens, ride in the grid of hta_bwd_dkdv.h).
#pragma once
#include "hta_common.h"
#include "hta_mfma.h"
#include "hta_rows.h"
#include "hta_tiles.h"

namespace hta {
namespace {

constexpr int BRIEF_NW = 4;  // waves of a workgroup

template <int D, bool RT>
struct Brief {
    static constexpr int TILE = 32 * D;              // elements of a 32-row tile
    static constexpr int CPR = D / 8;                // 16-byte chunks per row
    static constexpr int RPC = 64 / CPR;             // rows per 1 KB copy
    static constexpr int CPT = 32 / RPC;             // copies per tile
    // dK/dV: Q, dO, -lse/scale[32], -delta[32] of a unit; with real-time tokens also the rows' limits, int[32] (written twice)
    static constexpr int UNIT_BYTES = 2 * TILE * 2 + 256 + (RT ? 256 : 0);
    static constexpr int KV_BYTES = 2 * TILE * 2;    // dQ: K, V of a block
    static constexpr int SLOTS = 2;
    static constexpr int KEY_PITCH = D + 4, ROW_PITCH = D + 4;                 // floats per row of the final sums
    static constexpr int SUM_BYTES = BRIEF_NW * 32 * 2 * KEY_PITCH * 4;             // dK and dV of every wave
    static constexpr int RING_BYTES = BRIEF_NW * SLOTS * UNIT_BYTES;
    static constexpr int BYTES = RING_BYTES > SUM_BYTES ? RING_BYTES : SUM_BYTES;
};

// ---------------------------------------------------------------------------------------- dK, dV
// TAIL: only users with real-time tokens, and of those only the 32-key blocks behind the last whole block of history keys.  Most
// rows of a user see none of those keys; the units of such rows are skipped.
// WAYS: waves that share the rows of a 32-key block and add up their sums; a workgroup has BRIEF_NW / WAYS such blocks.
template <int D, int WAYS, bool RT, bool PW, bool TAIL = false>
__device__ __forceinline__ void brief_dkdv(const Params& p, const RowMap& map, unsigned id, int n_kt, int spread, unsigned char* smem) {
    using BR = Brief<D, RT>;
    constexpr int NKS = D / 16, NDB = D / 32, CPT = BR::CPT;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const WorkItem w = decode_spread(id, p.batch * p.Hkv, p.Hkv, n_kt, spread);
    if (!w.valid) return;
    const int b = scheduled_user(p, w.user_slot), g = w.y, r = p.Hq / p.Hkv;
    const int L = p.hist_len[b], T = p.n_targets[b];
    const int64_t q_base = p.q_off[b], kv_base = p.kv_off[b];
    const int LK = L + (RT ? p.rt_len[b] : 0);  // keys that receive gradient here: history, then real-time
    if (TAIL && LK == L) return;  // (a user without real-time tokens is bwd_dkdv_kernel's alone, bit for bit as in a call without any)
    constexpr int KBS = BRIEF_NW / WAYS;
    const int key0 = w.tile * (KBS * 32) + (TAIL ? L & ~31 : 0);
    if (key0 >= LK) return;  // uniform for the workgroup
    const int way = wave % WAYS, kw = key0 + wave / WAYS * 32;
    const int n_rows = p.layer == 0 ? LK + T : T, tok_shift = p.layer == 0 ? 0 : LK;
    const int tiles = (n_rows + map.rows - 1) / map.rows, n_units = tiles * map.n_chunks;  // unit = (row tile, head chunk)
    const int n_mine = kw < LK && n_units > way ? (n_units - way + WAYS - 1) / WAYS : 0;
    const float c2 = p.scale * LOG2E;
    const bool key_live = kw + l32 < LK;
    const bool masked = kw + 32 > L;  // ragged, or (RT) among the real-time keys

    // Copies of a unit: lane constants for the rows this lane fetches (packed row rho of the unit -> row q, head hh)
    uint32_t voff[CPT];
    int crow[CPT];  // row inside the unit of the lane's chunk in copy j; a lane that stands for no row repeats row 0
#pragma unroll
    for (int j = 0; j < CPT; j++) {
        const int trow = j * BR::RPC + lane / BR::CPR;
        int q = (int)(((uint32_t)trow * map.magic) >> 20), hh = trow - q * map.heads;
        if (q >= map.rows) q = 0, hh = 0;
        crow[j] = q;
        voff[j] = (uint32_t)(((q * p.Hq + hh) * D + (((lane % BR::CPR) ^ swizzle<D>(trow)) << 3)) * 2);
    }
    const int sq = (int)(((uint32_t)l32 * map.magic) >> 20), sh = l32 - sq * map.heads;  // the row whose statistics the lane fetches
    const uint32_t lds0 = lds_address(smem) + (uint32_t)wave * BR::SLOTS * BR::UNIT_BYTES;
    const bool even = map.rows * map.heads == 32 && r % map.heads == 0;  // no lane without a row, no chunk without a head
    auto issue = [&](int i) __attribute__((always_inline)) {
        if (i >= n_mine) return;
        const int u = way + i * WAYS;
        const int chunk = map.n_chunks == 1 ? 0 : u % map.n_chunks, row0 = (map.n_chunks == 1 ? u : u / map.n_chunks) * map.rows;
        const int h0 = g * r + chunk * map.heads, n_heads = min(map.heads, r - chunk * map.heads);
        const uint32_t dst = lds0 + (uint32_t)(i & 1) * BR::UNIT_BYTES;
        const int64_t base = ((q_base + row0) * p.Hq + h0) * (int64_t)D;
        const bool whole = even && row0 + map.rows <= n_rows;
        const __bf16* qb = (const __bf16*)p.q + base;
        const __bf16* db = (const __bf16*)p.dout + base;
#pragma unroll
        for (int j = 0; j < CPT; j++) {
            uint32_t off = voff[j];
            if (!whole) {  // rows past the end and heads past the group repeat row 0, head h0 of the unit, with no weight
                const int trow = j * BR::RPC + lane / BR::CPR;
                const int hh = trow - (int)(((uint32_t)trow * map.magic) >> 20) * map.heads;
                if (row0 + crow[j] >= n_rows || hh >= n_heads) off = (uint32_t)((((lane % BR::CPR) ^ swizzle<D>(trow)) << 3) * 2);
            }
            copy16_global_to_lds_at(qb, off, dst + j * 1024);
            copy16_global_to_lds_at(db, off, dst + BR::TILE * 2 + j * 1024);
        }
        // likewise the statistics: of row 0, head h0, where there is no row (see row_start)
        const bool live = whole || (row0 + sq < n_rows && sq < map.rows && sh < n_heads);
        const int row = row0 + (live ? sq : 0), h = h0 + (live ? sh : 0);
        copy4_global_to_lds_at(row_start(p, hf, (int64_t)h * p.total_q + q_base + row, live), dst + 4 * BR::TILE);
        if constexpr (RT) copy4_global_to_lds_at(p.lim + q_base + row, dst + 4 * BR::TILE + 256);
    };
    constexpr int COPIES = 2 * CPT + 1 + (RT ? 1 : 0);
    issue(0);
    issue(1);

    int nat[NKS], tlo[NDB], thi[NDB];
    natural_offsets<D>(nat, lane);
    transposed_offsets<D>(tlo, thi, lane);
    // stationary operands: K and V rows of the workgroup's keys (B operand of S = Q K^T and dP = dO V^T)
    bf16x8 kf[NKS], vf[NKS];
    {
        const int key = min(kw + l32, LK - 1);
        const int64_t off = ((kv_base + key) * p.Hkv + g) * D + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            kf[ks] = *(const bf16x8*)((const __bf16*)p.k + off + ks * 16);
            vf[ks] = *(const bf16x8*)((const __bf16*)p.v + off + ks * 16);
        }
    }
    floatx16 dK[NDB], dV[NDB];  // transposed: [d (registers)][key (lanes)]
#pragma unroll
    for (int db = 0; db < NDB; db++)
#pragma unroll
        for (int v = 0; v < 16; v++) dK[db][v] = 0.f, dV[db][v] = 0.f;
    wait_vmem_loads();  // from here on the only vector-memory traffic of the loop are the copies

    auto unit = [&](int i, auto Masked) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(Masked)::value;
        if (i + 1 < n_mine) wait_vmem_outstanding<COPIES>(); else wait_vmem_outstanding<0>();
        const __bf16* Qs = (const __bf16*)(smem + (wave * BR::SLOTS + (i & 1)) * BR::UNIT_BYTES);
        const __bf16* dOs = Qs + BR::TILE;
        const float* ss = (const float*)(dOs + BR::TILE);
        const int u0 = way + i * WAYS, own0 = tok_shift + (map.n_chunks == 1 ? u0 : u0 / map.n_chunks) * map.rows;  // token of the unit's first row
        if constexpr (MASKED && RT && D < 128) {  // (at 128 the branch costs more registers than there are)
            const bool sees = ((const int*)(ss + 64))[l32] > kw || (own0 + map.rows > kw && own0 < kw + 32);
            if (__builtin_amdgcn_ballot_w64(sees) == 0) {  // no row of the unit sees a key of this block
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                issue(i + 2);
                return;
            }
        }
        floatx16 S, dP;  // [row (registers)][key (lanes)], starting from -lse/scale and -delta of their rows
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const floatx4 l4 = *(const floatx4*)(ss + 8 * j + 4 * hf), d4 = *(const floatx4*)(ss + 32 + 8 * j + 4 * hf);
#pragma unroll
            for (int e = 0; e < 4; e++) S[4 * j + e] = l4[e], dP[4 * j + e] = d4[e];
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            S = mfma32(*(const bf16x8*)(Qs + nat[ks]), kf[ks], S);
            dP = mfma32(*(const bf16x8*)(dOs + nat[ks]), vf[ks], dP);
        }
        bf16x8 dot[NDB][2], qt[NDB][2];
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) {
                dot[db][s2] = lds_read_tr_pair(dOs + tlo[db] + 16 * s2 * D, dOs + thi[db] + 16 * s2 * D);
                qt[db][s2] = lds_read_tr_pair(Qs + tlo[db] + 16 * s2 * D, Qs + thi[db] + 16 * s2 * D);
            }
        int limv[16];
        if constexpr (MASKED && RT) {
            typedef int int4v __attribute__((ext_vector_type(4)));
            const int* ls = (const int*)(ss + 64);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int4v l4 = *(const int4v*)(ls + 8 * j + 4 * hf);
#pragma unroll
                for (int e = 0; e < 4; e++) limv[4 * j + e] = l4[e];
            }
        }
        bf16x8 pb[2], dsb[2];
        static_for<0, 16>([&](auto V) {
            constexpr int v = decltype(V)::value;
            bool vis = true;
            if constexpr (MASKED && RT) {  // below the row's limit, or the row's own token (the own key of a real-time row)
                const int rho = 8 * (v / 4) + 4 * hf + (v % 4);
                vis = kw + l32 < limv[v] || (key_live && kw + l32 == own0 + (int)(((uint32_t)rho * map.magic) >> 20));
            } else if constexpr (MASKED) {
                vis = key_live;
            }
            float pw, sp;
            if constexpr (PW) {
                const float sg = pw_sigmoid(S[v], -c2);
                pw = pw_silu(S[v], sg);  // P / scale
                sp = pw_silu_prime_of(pw, sg, p.scale);
                if constexpr (MASKED) sp = vis ? sp : 0.f;
            } else {
                pw = fast_exp2(S[v] * c2);
            }
            if constexpr (MASKED) pw = vis ? pw : 0.f;
            if constexpr (!PW) sp = pw;
            pb[v / 8][v % 8] = (__bf16)pw;
            dsb[v / 8][v % 8] = (__bf16)(sp * dP[v]);
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read
        issue(i + 2);
        // dV^T[d][key] += dO^T[d][row] P[row][key];  dK^T[d][key] += Q^T[d][row] dS[row][key]
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) {
                dV[db] = mfma32(dot[db][s2], pb[s2], dV[db]);
                dK[db] = mfma32(qt[db][s2], dsb[s2], dK[db]);
            }
    };
    if (masked) {
        for (int i = 0; i < n_mine; i++) unit(i, std::true_type{});
    } else {
        for (int i = 0; i < n_mine; i++) unit(i, std::false_type{});
    }

    // add up the sums of the waves of each key block (a lane has its key's row, in words of 16 bytes); rows of 16 bytes per thread go out
    lds_barrier();
    float* acc = (float*)smem;  // [wave][dK, dV][key][KEY_PITCH]
    constexpr int WAVE_FLOATS = 2 * 32 * BR::KEY_PITCH;
    {
        float* o = acc + wave * WAVE_FLOATS + l32 * BR::KEY_PITCH + 4 * hf;
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int v4 = 0; v4 < 4; v4++) {
                *(floatx4*)(o + db * 32 + 8 * v4) = floatx4{dK[db][4 * v4], dK[db][4 * v4 + 1], dK[db][4 * v4 + 2], dK[db][4 * v4 + 3]};
                *(floatx4*)(o + 32 * BR::KEY_PITCH + db * 32 + 8 * v4) = floatx4{dV[db][4 * v4], dV[db][4 * v4 + 1], dV[db][4 * v4 + 2], dV[db][4 * v4 + 3]};
            }
    }
    lds_barrier();
    constexpr int OCTS = D / 8;
    for (int e = tid; e < KBS * 2 * 32 * OCTS; e += BRIEF_NW * 64) {
        const int c = e % OCTS, row = e / OCTS % 64, kb = e / OCTS / 64;  // rows 0..31: dK, 32..63: dV
        const int key = key0 + kb * 32 + (row & 31);
        if (key >= LK) continue;
        const float* a = acc + kb * WAYS * WAVE_FLOATS + row * BR::KEY_PITCH + 8 * c;
        floatx4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
        for (int k = 0; k < WAYS; k++) {
            lo += *(const floatx4*)(a + k * WAVE_FLOATS);
            hi += *(const floatx4*)(a + k * WAVE_FLOATS + 4);
        }
        const float f = PW ? p.scale * p.norm : row < 32 ? p.scale : 1.f;
        bf16x8 o8;
#pragma unroll
        for (int j = 0; j < 4; j++) o8[j] = (__bf16)(lo[j] * f), o8[4 + j] = (__bf16)(hi[j] * f);
        *(bf16x8*)((__bf16*)(row < 32 ? p.dk : p.dv) + ((kv_base + key) * p.Hkv + g) * D + 8 * c) = o8;
    }
}

}  // namespace
}  // namespace hta
