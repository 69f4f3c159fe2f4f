// The dK/dV pass of the bf16 backward (gfx950): kernel templates and their launchers, included by the translation
// units that instantiate them (hta_bwd_bf16.hip: all but those of head_dim 128 with softmax weights, which
// hta_bwd_dkdv128_bf16.hip compiles with another instruction scheduling strategy, see build.py).
//
//   bwd_dkdv: key-stationary: a wave owns 32 history keys (K, V fragments and the dK, dV accumulators
//      stay in registers for the whole kernel), the workgroup streams (head, 32-row block) tiles of Q
//      and dO through LDS, shared by its waves.  S = Q K^T and dP = dO V^T have the key on the lane, so
//      P and dS in accumulator layout are directly the k-operand of dV = P^T dO and dK = dS^T Q.
//      dk/dv of history keys are written once.
#pragma once
#include "../../include/mtfm_hta.h"
#include "hta_common.h"
#include "hta_dkdv_brief.h"
#include "hta_mfma.h"
#include "hta_tiles.h"

namespace hta {
namespace {

// ---------------------------------------------------------------------------------------- dK, dV
template <int D, int NW>
struct DkdvSmem {
    static constexpr int UPI = 2;      // (head, 32-row block) units per loop iteration, i.e. per workgroup barrier
    static constexpr int NSTAGE = 3;   // iterations resident in LDS: one being consumed, two in flight
    static constexpr int TILE = 32 * D;                 // one unpadded, swizzled 32-row tile (elements)
    static constexpr size_t UNIT_BYTES = (size_t)2 * TILE * 2 + 2 * 32 * sizeof(float);  // Q, dO, -lse/scale[32], -delta[32]
    static constexpr size_t STAGE_BYTES = UPI * UNIT_BYTES;
    static constexpr size_t BYTES = NSTAGE * STAGE_BYTES;
};

// One workgroup per (user, kv head, tile of NW*32 history keys).  Q and dO tiles travel global -> LDS directly
// (no register stop-over), two iterations ahead of their use.
// Of a user with real-time tokens (mask rule 2) these workgroups take the whole 32-key blocks of the history only, which every
// row sees: no mask.  The blocks behind them (TAILS: the last blocks of the grid, behind the persistent ones; at
// d = 128, where both in one kernel do not fit the registers, a launch of their own) are
// brief_dkdv's, whose masked stream skips the rows that see none of their keys; they fill the units that run out of
// history.  (256 users of 512..1024 + 32..128 + 64 tokens: 899 us, against 954 with one masked instruction stream for all
// keys and the rows' limits staged next to every unit.)
// PW: the pointwise reading of phi2 -- P = silu(scale S), dS = dP o silu'(scale S); the staged row statistics are
// zeros for rows that exist (the sentinel for rows that do not still removes them), norm is applied at the store.
template <int D, int NW, bool TAILS, bool PW = false>
__global__ __launch_bounds__(NW * 64, D > 64 ? 1 : 2) void bwd_dkdv_kernel(Params p, int tpg, int spread, unsigned per_xcd, unsigned n_persistent,
                                                                       RowMap map, int tail_tpg) {
    using SM = DkdvSmem<D, NW>;
    constexpr int UPI = SM::UPI, NSTAGE = SM::NSTAGE;
    constexpr int NKS = D / 16, NDB = D / 32;
    constexpr int CPR = D / 8;                  // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;               // rows covered by one wave-wide 1 KB copy
    constexpr int IPT = 32 / RPI;               // copies per tile
    constexpr int IPW = (IPT + NW - 1) / NW;    // copies per tile issued by one wave (the last may be idle)
    constexpr int COPIES = UPI * 2 * IPW;       // direct copies per wave and iteration (when the wave takes part)
    static_assert(IPT % NW == 0 || IPT < NW, "tile copies must split evenly over the waves");
    static_assert(UPI <= NW, "wave uu copies the row statistics of unit uu");
    constexpr size_t LDS_BYTES = TAILS && (size_t)Brief<D, true>::BYTES > SM::BYTES ? (size_t)Brief<D, true>::BYTES : SM::BYTES;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS_BYTES];
    auto stage_ptr = [&](auto St) -> unsigned char* { return smem + decltype(St)::value % 3 * SM::STAGE_BYTES; };
    static_assert(NSTAGE == 3, "three stages");
    if (TAILS && blockIdx.x >= n_persistent) {
        brief_dkdv<D, BRIEF_NW, true, PW, true>(p, map, blockIdx.x - n_persistent, tail_tpg, 0, smem);
        return;
    }

    __shared__ int s_item;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;

    // The next item is taken four to six iterations before the current one ends, early enough for the atomic to have returned by then.  (Taken with the
    // start of the current one, the last items of the lists waited behind items in progress while other workgroups left.  Whole steps: 256 users
    // of 512..1024 keys 1815 -> 1795 us, 238 of 366..732 930 -> 901, 28 of up to 7896 2827 -> 2514; at head_dim 128 33 users of 434 + 60
    // keys 584 -> 497, 23 of 715..2379 2749 -> 2496, 128 of 750..8192 50.2 -> 49.7 ms; of 40 sampled calls one 1 % slower.  Waited for in the loop
    // instead: 112 calls 1.000 of the time; backward passes of 128 users of 750..8192 keys 37.8 -> 38.0 ms, 180 of 300..900, 4/2 heads of 32, 203.1 -> 204.9 us.)
    const int xcd = blockIdx.x % N_XCD;
    unsigned taken = blockIdx.x / N_XCD;
    bool asked;
    auto ask = [&](unsigned& answer) __attribute__((always_inline)) {
        if (tid == 0) queue_ask(answer, p.queue, xcd, per_xcd, n_persistent);
        asked = true;
    };

    // one work item: a (user, kv head, key tile) triple
    auto process = [&](unsigned id) {
    unsigned answer;  // (an item's own: across the loop over items its register would be copied, which waits for every store of the item)
    asm volatile("" : "=v"(answer));
    const WorkItem w = decode_spread(id, p.batch * p.Hkv, p.Hkv, tpg, spread);
    if (!w.valid) return;
    const int b = scheduled_user(p, w.user_slot), g = w.y;
    const int L = p.hist_len[b], T = p.n_targets[b];
    const int R = p.rt_len ? p.rt_len[b] : 0;
    const int LK = R > 0 ? L & ~31 : L;  // keys that receive gradient here
    const int key0 = w.tile * (NW * 32);
    if (key0 >= LK) return;  // uniform: this key tile does not exist for the user
    const int n_rows = p.layer == 0 ? L + R + T : T;
    const int r = p.Hq / p.Hkv;
    const int64_t q_base = p.q_off[b], kv_base = p.kv_off[b];
    const float c2 = p.scale * LOG2E;
    const int kw = key0 + wave * 32;        // first key of this wave
    const bool wave_live = kw < LK;         // a wave past the last key only helps staging
    const bool key_live = kw + l32 < LK;
    const bool wave_ragged = kw + 32 > LK;  // past the end: masked instruction stream
    const bool copies = IPT >= NW || wave < IPT;   // does this wave issue tile copies?

    // per-lane element offsets into a swizzled tile
    int nat_off[NKS];   // row l32, chunk 2*ks + hf: fragments with the row on the lane
#pragma unroll
    for (int ks = 0; ks < NKS; ks++) nat_off[ks] = l32 * D + (((2 * ks + hf) ^ swizzle<D>(l32)) << 3);
    // transposed fragments: rows 4*hf + (lane%16)/4 and 8 below (+16 per k-step, which leaves the swizzle
    // unchanged), 4 elements at column 32*db + 16*((lane/16)%2) + 4*(lane%4)
    int tr_lo[NDB], tr_hi[NDB];
    {
        const int pl = lane & 15, trow = 4 * hf + (pl >> 2);
#pragma unroll
        for (int db = 0; db < NDB; db++) {
            const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((pl & 3) >> 1);
            tr_lo[db] = trow * D + ((chunk ^ swizzle<D>(trow)) << 3) + 4 * (pl & 1);
            tr_hi[db] = (trow + 8) * D + ((chunk ^ swizzle<D>(trow + 8)) << 3) + 4 * (pl & 1);
        }
    }

    // stationary operands: K and V rows of the wave's keys (B operand of S = Q K^T and dP = dO V^T)
    bf16x8 kf[NKS], vf[NKS];
    {
        const int key = key_live ? kw + l32 : LK - 1;
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
        for (int v = 0; v < 16; v++) {
            dK[db][v] = 0.f;
            dV[db][v] = 0.f;
        }

    const int n_rb = (n_rows + 31) / 32;
    const int n_units = n_rb * r;  // unit u = (32-row block u / r, head g*r + u % r)
    const int n_iter = (n_units + UPI - 1) / UPI;  // 0 for a user without query rows: dK = dV = 0 is still written

    // Q and dO tiles of iteration `it` -> stage it % NSTAGE.  Copy j of a tile covers rows j*RPI .. j*RPI+RPI-1:
    // lane i lands at chunk position i % CPR of row j*RPI + i / CPR, so it fetches the chunk that belongs there.
    // The calls come in the order it = 0, 1, 2, ...; the unit the next call starts with is kept in (iss_rb, iss_hh).
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    uint32_t tile_voff[IPW];  // byte offset of the lane's chunk from the first element of (row0, head h)
#pragma unroll
    for (int jj = 0; jj < IPW; jj++) {
        const int trow = (wave + jj * NW) * RPI + lane / CPR;
        tile_voff[jj] = (uint32_t)((trow * p.Hq * D + (((lane % CPR) ^ swizzle<D>(trow)) << 3)) * 2);
    }
    const float* stat_lane = (hf == 0 ? p.neg_lse_s : p.neg_delta) + q_base + l32;
    int iss_rb = 0, iss_hh = 0;
    auto issue_tiles = [&](auto St) {
        const uint32_t stage = lds_address(stage_ptr(St));
#pragma unroll
        for (int uu = 0; uu < UPI; uu++) {
            // a unit past the last one repeats the last one, with no weight
            const bool past = iss_rb >= n_rb;
            const int rb = past ? n_rb - 1 : iss_rb, hh = past ? r - 1 : iss_hh;
            const int row0 = rb * 32, h = g * r + hh;
            const bool whole = !past && row0 + 32 <= n_rows;  // every row exists: no per-lane address arithmetic
            const uint32_t unit = stage + uu * (uint32_t)SM::UNIT_BYTES;
            const int64_t ubase = ((q_base + row0) * p.Hq + h) * (int64_t)D;
            if (whole) {
#pragma unroll
                for (int jj = 0; jj < (copies ? IPW : 0); jj++) {
                    const uint32_t dst = unit + (uint32_t)(wave_u + jj * NW) * 1024u;
                    copy16_global_to_lds_at((const __bf16*)p.q + ubase, tile_voff[jj], dst);
                    copy16_global_to_lds_at((const __bf16*)p.dout + ubase, tile_voff[jj], dst + (uint32_t)SM::TILE * 2u);
                }
                if (wave_u == uu) copy4_global_to_lds_at(stat_lane + ((int64_t)h * p.total_q + row0), unit + 4u * (uint32_t)SM::TILE);
            } else {
#pragma unroll
                for (int jj = 0; jj < (copies ? IPW : 0); jj++) {
                    const int trow = (wave + jj * NW) * RPI + lane / CPR;
                    int row = row0 + trow;
                    row = row < n_rows ? row : n_rows - 1;  // rows past the end repeat the last row, with no weight
                    const int chunk = (lane % CPR) ^ swizzle<D>(trow);
                    const int64_t off = ((q_base + row) * p.Hq + h) * D + chunk * 8;
                    const uint32_t dst = unit + (uint32_t)(wave_u + jj * NW) * 1024u;
                    copy16_global_to_lds_at((const __bf16*)p.q + off, dst);
                    copy16_global_to_lds_at((const __bf16*)p.dout + off, dst + (uint32_t)SM::TILE * 2u);
                }
                // A row that does not exist starts from the sentinel behind the -lse/scale array, a huge negative
                // number: its weights P = exp(scale * that) are exactly 0, and so is all it would add to dK and dV.
                if (wave_u == uu) {
                    int row = row0 + l32;
                    const bool dead = past || row >= n_rows;
                    row = row < n_rows ? row : n_rows - 1;
                    copy4_global_to_lds_at(row_start(p, hf, (int64_t)h * p.total_q + q_base + row, !dead), unit + 4u * (uint32_t)SM::TILE);
                }
            }
            if (!past && ++iss_hh == r) {
                iss_hh = 0;
                iss_rb++;
            }
        }
    };
    // wait until at most the copies this wave has issued for its K most recent iterations are outstanding
    auto wait_all_but_iterations = [&](auto Kc) {
        constexpr int K = decltype(Kc)::value;
        const bool extra = wave < UPI;  // one more copy per iteration: statistics
        if (copies) {
            if (extra) wait_vmem_outstanding<K * (COPIES + 1)>(); else wait_vmem_outstanding<K * COPIES>();
        } else {
            if (extra) wait_vmem_outstanding<K>(); else wait_vmem_outstanding<0>();
        }
    };
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};

    // The wave's work on one (head, 32-row block) unit against its 32 keys, in four steps that the loop below
    // interleaves across units: fetch the operands, S and dP, the weights, the two accumulations.
    struct Operands {
        bf16x8 qa[NKS], da[NKS];
        floatx16 S, dP;  // [row (registers)][key (lanes)]
    };
    struct Transposed {
        bf16x8 dot[NDB][2], qt[NDB][2];
    };
    auto load_operands = [&](const unsigned char* ubase, Operands& o) {
        const __bf16* Qs = (const __bf16*)ubase;
        const __bf16* dOs = Qs + SM::TILE;
        const float* ss = (const float*)(dOs + SM::TILE);
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            o.qa[ks] = *(const bf16x8*)(Qs + nat_off[ks]);
            o.da[ks] = *(const bf16x8*)(dOs + nat_off[ks]);
        }
        // accumulators start from -lse/scale and -delta of their rows (registers 4j..4j+3 hold rows 8j+4hf .. +3)
        floatx4 l4[4], d4[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            l4[j] = *(const floatx4*)(ss + 8 * j + 4 * hf);
            d4[j] = *(const floatx4*)(ss + 32 + 8 * j + 4 * hf);
        }
        o.S = __builtin_shufflevector(__builtin_shufflevector(l4[0], l4[1], 0, 1, 2, 3, 4, 5, 6, 7),
                                      __builtin_shufflevector(l4[2], l4[3], 0, 1, 2, 3, 4, 5, 6, 7), 0, 1, 2, 3, 4, 5, 6, 7, 8,
                                      9, 10, 11, 12, 13, 14, 15);
        o.dP = __builtin_shufflevector(__builtin_shufflevector(d4[0], d4[1], 0, 1, 2, 3, 4, 5, 6, 7),
                                       __builtin_shufflevector(d4[2], d4[3], 0, 1, 2, 3, 4, 5, 6, 7), 0, 1, 2, 3, 4, 5, 6, 7,
                                       8, 9, 10, 11, 12, 13, 14, 15);
    };
    auto scores = [&](Operands& o) {
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            o.S = mfma32(o.qa[ks], kf[ks], o.S);     // S - lse/scale
            o.dP = mfma32(o.da[ks], vf[ks], o.dP);   // dP - delta
        }
    };
    auto load_transposed = [&](const unsigned char* ubase, Transposed& f) {
        const __bf16* Qs = (const __bf16*)ubase;
        const __bf16* dOs = Qs + SM::TILE;
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) {
                f.dot[db][s2] = lds_read_tr_pair(dOs + tr_lo[db] + 16 * s2 * D, dOs + tr_hi[db] + 16 * s2 * D);
                f.qt[db][s2] = lds_read_tr_pair(Qs + tr_lo[db] + 16 * s2 * D, Qs + tr_hi[db] + 16 * s2 * D);
            }
    };
    struct Weights {
        bf16x8 pb[2], dsb[2];
    };
    auto weights = [&](const Operands& o, Weights& wt, auto ragged) {
        constexpr bool MASKED = decltype(ragged)::value;
        if constexpr (PW) {
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const float sg = pw_sigmoid(o.S[v], -c2);
                float pw = pw_silu(o.S[v], sg), sp = pw_silu_prime_of(pw, sg, p.scale);  // P / scale
                if constexpr (MASKED) {  // keys past the history carry no weight
                    pw = key_live ? pw : 0.f;
                    sp = key_live ? sp : 0.f;
                }
                wt.pb[v / 8][v % 8] = (__bf16)pw;
                wt.dsb[v / 8][v % 8] = (__bf16)(sp * o.dP[v]);
            }
            return;
        }
#pragma unroll
        for (int v = 0; v < 16; v++) {
            float pw = fast_exp2(o.S[v] * c2);
            if constexpr (MASKED) {
                pw = key_live ? pw : 0.f;  // keys past the history carry no weight
            }
            wt.pb[v / 8][v % 8] = (__bf16)pw;
            wt.dsb[v / 8][v % 8] = (__bf16)(pw * o.dP[v]);
        }
    };
    // dV^T[d][key] += dO^T[d][row] P[row][key];  dK^T[d][key] += Q^T[d][row] dS[row][key]
    auto accumulate = [&](const Weights& wt, const Transposed& f) {
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) {
                dV[db] = mfma32(f.dot[db][s2], wt.pb[s2], dV[db]);
                dK[db] = mfma32(f.qt[db][s2], wt.dsb[s2], dK[db]);
            }
    };

    const std::integral_constant<int, 0> st0{};
    const std::integral_constant<int, 1> st1{};
    const std::integral_constant<int, 2> st2{};
    static_assert(UPI == 2, "the loop below is written out for two units per iteration");
    // prologue: all three stages requested while the K/V fragments are still on their way (one memory latency instead
    // of two at the start of every item).  From the wait on, the only vector-memory traffic of the loop are the
    // asynchronous copies, which this code counts itself, and wave 0's request for the next item, which makes one or two of
    // its counted waits reach a copy further; the compiler must not be left with pending loads of its own that it would
    // wait for inside the loop.
    if (n_iter > 0) issue_tiles(st0);
    if (n_iter > 1) issue_tiles(st1);
    if (n_iter > 2) issue_tiles(st2);
    wait_vmem_loads();
    lds_barrier();

    // Iteration `it` consumes stage it % 3.  Its barrier sits in the middle of the second unit, after the last LDS read
    // of the stage: behind it the stage is refilled for iteration it+3 and the operands of iteration it+1 are fetched,
    // both while the second unit's accumulations keep the matrix unit busy.
    auto run = [&](auto ragged) {
        Operands cur;
        load_operands(stage_ptr(st0), cur);
        auto iteration = [&](int it, auto St) {
            constexpr int st = decltype(St)::value;
            const unsigned char* base = stage_ptr(St);
            Operands nxt;
            Transposed f;
            Weights wt;
            // The second unit's S and dP are requested before the first unit's weights are formed, and the first
            // unit's accumulations come after the second unit's weights: each block of vector work then has matrix
            // instructions of the other unit in the stream around it (3 % at d = 64, 6 % at d = 128).
            Weights wt0;
            scores(cur);
            load_operands(base + SM::UNIT_BYTES, nxt);
            weights(cur, wt0, ragged);
            scores(nxt);
            load_transposed(base, f);
            weights(nxt, wt, ragged);
            accumulate(wt0, f);
            load_transposed(base + SM::UNIT_BYTES, f);
            // copies of iteration it+1 must have landed; those of it+2 may stay in flight
            if (it + 2 < n_iter) wait_all_but_iterations(c1); else wait_all_but_iterations(c0);
            lds_barrier();
            if (it + 3 < n_iter) issue_tiles(St);
            // (behind the last iteration this reads a stage that holds nothing new; the values are not used)
            load_operands(stage_ptr(std::integral_constant<int, (st + 1) % 3>{}), cur);
            accumulate(wt, f);
        };
        for (int it = 0; it < n_iter; it += 3) {
            if (it + 6 >= n_iter && !asked) ask(answer);
            iteration(it, st0);
            if (it + 1 < n_iter) iteration(it + 1, st1);
            if (it + 2 < n_iter) iteration(it + 2, st2);
        }
    };
    // a wave past the history only helps staging: same waits, same barriers, same copies
    auto run_idle = [&]() {
        auto iteration = [&](int it, auto St) {
            if (it + 2 < n_iter) wait_all_but_iterations(c1); else wait_all_but_iterations(c0);
            lds_barrier();
            if (it + 3 < n_iter) issue_tiles(St);
        };
        for (int it = 0; it < n_iter; it += 3) {
            iteration(it, st0);
            if (it + 1 < n_iter) iteration(it + 1, st1);
            if (it + 2 < n_iter) iteration(it + 2, st2);
        }
    };
    if (n_iter > 0) {
        if (!wave_live) run_idle();
        else if (wave_ragged) run(std::true_type{});
        else run(std::false_type{});
    }
    if (asked) taken = queue_answer(answer, xcd, per_xcd, n_persistent);

    // A lane writes its key's row, 16 bytes at a time.  (The other way round the products leave keys in registers and features on the lanes, and
    // each store has 2 bytes per lane: 128 of them at head_dim 128, 2.5 us of an item.  Whole steps, this and its like in the other kernels: 256 users of
    // 512..1024 keys 1783 -> 1743 us, 64 of 128..512 145.0 -> 140.0, 246 of 28..115 + 8..70 real-time tokens at head_dim 128 836 -> 795.)
    if (wave_live && key_live) {
        const int64_t off = ((kv_base + kw + l32) * p.Hkv + g) * D + 8 * hf;
        static_for<0, 2 * NDB>([&](auto I) {
            constexpr int i = decltype(I)::value;
            *(bf16x8*)((__bf16*)p.dk + off + 16 * i) = rows_of_16<i % 2>(dK[i / 2], PW ? p.scale * p.norm : p.scale);
            *(bf16x8*)((__bf16*)p.dv + off + 16 * i) = rows_of_16<i % 2>(dV[i / 2], PW ? p.scale * p.norm : 1.f);
        });
    }
    };  // process

    // persistent workgroup: its own index first, then what the work counters give until all lists are exhausted
    for (;;) {
        if (__builtin_amdgcn_readfirstlane(tid >> 6) == 0) s_item = queue_resolve(p.queue, xcd, taken, per_xcd, n_persistent);
        __syncthreads();
        const int id = s_item;
        if (id < 0) break;
        asked = false;
        process((unsigned)id);
        if (!asked) {  // (no such item, or a wave that only helped staging)
            unsigned answer;
            asm volatile("" : "=v"(answer));
            ask(answer);
            taken = queue_answer(answer, xcd, per_xcd, n_persistent);
        }
        __syncthreads();  // the stages and s_item are free again
    }
}

// ---------------------------------------------------------------------------------------- dK, dV: few query rows
// The same pass for batches whose users have few query rows (a target-only layer: the candidates of a user against a
// long history).  bwd_dkdv_kernel streams the rows of a user past every 128-key tile again; with a handful of row
// blocks that is a prologue, a drained pipeline and an epilogue around four to eight iterations.  Here a workgroup
// takes a whole (user, kv head): it stages ALL (head, 32-row block) units of Q and dO in LDS once (at most MAX_UNITS of
// them, which is what the host checks), and then its waves walk the keys, 32 per wave and pass, each on its own: K/V
// fragments from global memory, every unit from LDS, dK/dV stored -- no barrier, no copy and no counted wait inside the
// key loop, and waves that drift apart.  Twelve waves, three per SIMD, one unit in flight per wave (168 registers, 17 more in scratch):
// measured against eight waves with two units interleaved per wave, as bwd_dkdv_kernel does it, the third wave hides
// more than the interleaving (dK/dV of a 512 x 2048 x 128 target layer 1.21 against 1.30 ms; streaming kernel 1.33).
// Softmax weights without real-time tokens only (the callers that need the other readings take the streaming kernel).  Most such
// calls now go through in one pass (hta_bwd_onepass_bf16.hip); left here are mostly those whose query heads per kv head are no power of two.
// There it is worth its place: of 562 calls that take it (3 to 16 query heads per kv head, 512..4000 keys, 256..3000 items) the whole backward
// is 1.08 times as fast on average as with the next best form (3 heads: 1.09, 6: 1.09, 12: 1.17; 870 users of up to 1764 keys x 31,
// 12/2 heads, 816 -> 626 us; at most 0.77 times, on little more than 256 items of unlike lengths).
template <int D, int NW>
struct DkdvResident {
    static constexpr int MAX_UNITS = 16;
    static constexpr int TILE = 32 * D;                                          // elements of a 32-row tile
    static constexpr size_t UNIT_BYTES = (size_t)2 * TILE * 2 + 2 * 32 * sizeof(float);  // Q, dO, -lse/scale[32], -delta[32]
    static constexpr size_t BYTES = MAX_UNITS * UNIT_BYTES;
};

template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 3) void bwd_dkdv_resident_kernel(Params p, unsigned per_xcd) {
    using SM = DkdvResident<D, NW>;
    constexpr int NKS = D / 16, NDB = D / 32;
    constexpr int CPR = D / 8;      // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;   // rows covered by one wave-wide 1 KB copy
    constexpr int IPT = 32 / RPI;   // copies per tile
    __shared__ __attribute__((aligned(1024))) unsigned char units[SM::BYTES];
    __shared__ int s_item;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int r = p.Hq / p.Hkv;
    const float c2 = p.scale * LOG2E;

    // per-lane element offsets into a swizzled tile (as in bwd_dkdv_kernel)
    int nat_off[NKS], tr_lo[NDB], tr_hi[NDB];
    natural_offsets<D>(nat_off, lane);
    transposed_offsets<D>(tr_lo, tr_hi, lane);
    // copy j of a tile covers rows j*RPI .. j*RPI+RPI-1: byte offset of the lane's chunk from (row0, head h)
    uint32_t tile_voff[IPT];
#pragma unroll
    for (int j = 0; j < IPT; j++) {
        const int trow = j * RPI + lane / CPR;
        tile_voff[j] = (uint32_t)((trow * p.Hq * D + (((lane % CPR) ^ swizzle<D>(trow)) << 3)) * 2);
    }

    struct Operands {
        bf16x8 qa[NKS], da[NKS];
        floatx16 S, dP;  // [row (registers)][key (lanes)]
    };
    struct Transposed {
        bf16x8 dot[NDB][2], qt[NDB][2];
    };
    struct Weights {
        bf16x8 pb[2], dsb[2];
    };

    // The next item is taken with the first wave's last pass over the keys (not with the item's start, see bwd_dkdv_kernel: 24 calls of 150 to 700
    // users 0.992 of the time of a step, 273 users of 2656 keys x 57, 12/4 heads, 946 -> 914 us, none slower by a hundredth).
    const int xcd = blockIdx.x % N_XCD;
    __shared__ unsigned s_taken;  // (a register would be one in scratch)
    if (tid == 0) s_taken = blockIdx.x / N_XCD;
    bool asked;
    auto ask = [&]() __attribute__((always_inline)) {
        if (tid == 0) s_taken = queue_take_ahead(p.queue, xcd, per_xcd, gridDim.x);
        asked = true;
    };

    auto process = [&](unsigned id) {
        const WorkItem w = decode_work(id, p.batch * p.Hkv, p.Hkv, 1);
        if (!w.valid) return;
        const int b = scheduled_user(p, w.user_slot), g = w.y;
        const int LK = p.hist_len[b], T = p.n_targets[b];
        if (LK <= 0) return;  // no key receives a gradient here
        const int n_rows = p.layer == 0 ? LK + T : T;
        const int n_rb = (n_rows + 31) / 32;
        // unit u = (32-row block u / r, head g*r + u % r).  (The launch is chosen from the caller's bounds on the rows of a
        // user; should a user exceed them, the clamp keeps the staging inside LDS.)
        const int n_units = min(n_rb * r, SM::MAX_UNITS);
        const int64_t q_base = p.q_off[b], kv_base = p.kv_off[b];

        // ---- stage every unit: wave u % NW brings unit u (2 * IPT tile copies and the row statistics)
        const uint32_t lds0 = lds_address(units);
        for (int u = wave_u; u < n_units; u += NW) {
            const int rb = u / r, h = g * r + u % r, row0 = rb * 32;
            const uint32_t unit = lds0 + (uint32_t)u * (uint32_t)SM::UNIT_BYTES;
            const bool whole = row0 + 32 <= n_rows;  // every row exists: no per-lane address arithmetic
            if (whole) {
                const int64_t ubase = ((q_base + row0) * p.Hq + h) * (int64_t)D;
#pragma unroll
                for (int j = 0; j < IPT; j++) {
                    copy16_global_to_lds_at((const __bf16*)p.q + ubase, tile_voff[j], unit + (uint32_t)j * 1024u);
                    copy16_global_to_lds_at((const __bf16*)p.dout + ubase, tile_voff[j], unit + (uint32_t)SM::TILE * 2u + (uint32_t)j * 1024u);
                }
                const float* stat = (hf == 0 ? p.neg_lse_s : p.neg_delta) + ((int64_t)h * p.total_q + q_base + row0 + l32);
                copy4_global_to_lds_at(stat, unit + 4u * (uint32_t)SM::TILE);
            } else {
#pragma unroll
                for (int j = 0; j < IPT; j++) {
                    const int trow = j * RPI + lane / CPR;
                    int row = row0 + trow;
                    row = row < n_rows ? row : n_rows - 1;  // rows past the end repeat the last row, with no weight
                    const int chunk = (lane % CPR) ^ swizzle<D>(trow);
                    const int64_t off = ((q_base + row) * p.Hq + h) * D + chunk * 8;
                    copy16_global_to_lds_at((const __bf16*)p.q + off, unit + (uint32_t)j * 1024u);
                    copy16_global_to_lds_at((const __bf16*)p.dout + off, unit + (uint32_t)SM::TILE * 2u + (uint32_t)j * 1024u);
                }
                // a row that does not exist starts from the sentinel behind the -lse/scale array: P = 0 exactly
                int row = row0 + l32;
                const bool dead = row >= n_rows;
                row = row < n_rows ? row : n_rows - 1;
                copy4_global_to_lds_at(row_start(p, hf, (int64_t)h * p.total_q + q_base + row, !dead), unit + 4u * (uint32_t)SM::TILE);
            }
        }
        wait_vmem_loads();
        lds_barrier();

        auto unit_ptr = [&](int u) { return units + (size_t)u * SM::UNIT_BYTES; };
        // ---- the keys, 32 per wave and pass
        for (int k0 = wave * 32; k0 < LK; k0 += NW * 32) {
            const int kw = k0;
            const bool key_live = kw + l32 < LK;
            const bool ragged = kw + 32 > LK;
            bf16x8 kf[NKS], vf[NKS];
            {
                const int key = key_live ? kw + l32 : LK - 1;
                const int64_t off = ((kv_base + key) * p.Hkv + g) * D + 8 * hf;
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    kf[ks] = *(const bf16x8*)((const __bf16*)p.k + off + ks * 16);
                    vf[ks] = *(const bf16x8*)((const __bf16*)p.v + off + ks * 16);
                }
            }
            // (behind the loads, which the wave waits for anyway, as it does for this)
            if (wave_u == 0 && k0 + NW * 32 >= LK) ask();
            floatx16 dK[NDB], dV[NDB];  // transposed: [d (registers)][key (lanes)]
#pragma unroll
            for (int db = 0; db < NDB; db++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    dK[db][v] = 0.f;
                    dV[db][v] = 0.f;
                }
            auto load_operands = [&](const unsigned char* ubase, Operands& o) {
                const __bf16* Qs = (const __bf16*)ubase;
                const __bf16* dOs = Qs + SM::TILE;
                const float* ss = (const float*)(dOs + SM::TILE);
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    o.qa[ks] = *(const bf16x8*)(Qs + nat_off[ks]);
                    o.da[ks] = *(const bf16x8*)(dOs + nat_off[ks]);
                }
                // accumulators start from -lse/scale and -delta of their rows (registers 4j..4j+3 hold rows 8j+4hf .. +3)
                floatx4 l4[4], d4[4];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    l4[j] = *(const floatx4*)(ss + 8 * j + 4 * hf);
                    d4[j] = *(const floatx4*)(ss + 32 + 8 * j + 4 * hf);
                }
                o.S = __builtin_shufflevector(__builtin_shufflevector(l4[0], l4[1], 0, 1, 2, 3, 4, 5, 6, 7),
                                              __builtin_shufflevector(l4[2], l4[3], 0, 1, 2, 3, 4, 5, 6, 7), 0, 1, 2, 3, 4, 5, 6,
                                              7, 8, 9, 10, 11, 12, 13, 14, 15);
                o.dP = __builtin_shufflevector(__builtin_shufflevector(d4[0], d4[1], 0, 1, 2, 3, 4, 5, 6, 7),
                                               __builtin_shufflevector(d4[2], d4[3], 0, 1, 2, 3, 4, 5, 6, 7), 0, 1, 2, 3, 4, 5, 6,
                                               7, 8, 9, 10, 11, 12, 13, 14, 15);
            };
            auto scores = [&](Operands& o) {
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    o.S = mfma32(o.qa[ks], kf[ks], o.S);     // S - lse/scale
                    o.dP = mfma32(o.da[ks], vf[ks], o.dP);   // dP - delta
                }
            };
            auto load_transposed = [&](const unsigned char* ubase, Transposed& f) {
                const __bf16* Qs = (const __bf16*)ubase;
                const __bf16* dOs = Qs + SM::TILE;
#pragma unroll
                for (int db = 0; db < NDB; db++)
#pragma unroll
                    for (int s2 = 0; s2 < 2; s2++) {
                        f.dot[db][s2] = lds_read_tr_pair(dOs + tr_lo[db] + 16 * s2 * D, dOs + tr_hi[db] + 16 * s2 * D);
                        f.qt[db][s2] = lds_read_tr_pair(Qs + tr_lo[db] + 16 * s2 * D, Qs + tr_hi[db] + 16 * s2 * D);
                    }
            };
            auto weights = [&](const Operands& o, Weights& wt) {
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    float pw = fast_exp2(o.S[v] * c2);
                    if (ragged) pw = key_live ? pw : 0.f;  // keys past the history carry no weight
                    wt.pb[v / 8][v % 8] = (__bf16)pw;
                    wt.dsb[v / 8][v % 8] = (__bf16)(pw * o.dP[v]);
                }
            };
            // dV^T[d][key] += dO^T[d][row] P[row][key];  dK^T[d][key] += Q^T[d][row] dS[row][key]
            auto accumulate = [&](const Weights& wt, const Transposed& f) {
#pragma unroll
                for (int db = 0; db < NDB; db++)
#pragma unroll
                    for (int s2 = 0; s2 < 2; s2++) {
                        dV[db] = mfma32(f.dot[db][s2], wt.pb[s2], dV[db]);
                        dK[db] = mfma32(f.qt[db][s2], wt.dsb[s2], dK[db]);
                    }
            };
            // one unit after the other: the other two waves of the SIMD fill what this one waits for
            {
                Operands cur;
                Transposed f;
                Weights wt;
                for (int u = 0; u < n_units; u++) {
                    load_operands(unit_ptr(u), cur);
                    scores(cur);
                    load_transposed(unit_ptr(u), f);
                    weights(cur, wt);
                    accumulate(wt, f);
                }
            }
            if (key_live) {
                const int64_t off = ((kv_base + kw + l32) * p.Hkv + g) * D + 8 * hf;
                static_for<0, 2 * NDB>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    *(bf16x8*)((__bf16*)p.dk + off + 16 * i) = rows_of_16<i % 2>(dK[i / 2], p.scale);
                    *(bf16x8*)((__bf16*)p.dv + off + 16 * i) = rows_of_16<i % 2>(dV[i / 2], 1.f);
                });
            }
        }
    };  // process

    // persistent workgroup, as in bwd_dkdv_kernel
    for (;;) {
        if (wave_u == 0) s_item = queue_resolve(p.queue, xcd, s_taken, per_xcd, gridDim.x);
        __syncthreads();
        const int id = s_item;
        if (id < 0) break;
        asked = false;
        process((unsigned)id);
        if (!asked) ask();  // (no such item, or one without keys)
        __syncthreads();  // the staged units and s_item are free again
    }
}

template <int D, bool PW>
__global__ __launch_bounds__(BRIEF_NW * 64, 1) void dkdv_tails_kernel(Params p, RowMap map, int tail_tpg) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[Brief<D, true>::BYTES];
    brief_dkdv<D, BRIEF_NW, true, PW, true>(p, map, blockIdx.x, tail_tpg, 0, smem);
}

// Spread of the lists (decode_spread): an XCD starts what is in its own list first, so where a few long users have much of the work their tiles
// go to four lists.  22 users of up to 4315 keys, 1413 in the mean, 16/2 heads of 128: whole step 3.48 -> 2.74 ms; 28 of up to 6611 keys, 8/2
// heads 2.39 -> 2.31; 20 of up to 6055 5.63 -> 5.43; five others of that kind within 1 %; the backward pass of 21 calls of 12 to 57 users with heavy
// tails 0.987, from 0.89 to 1.011.  Users alike, or many, gain nothing and read their operands into more L2s (256 users of 512..1024 keys 1806 -> 1825 us,
// 233 of up to 1195 3413 -> 3479).  The rule sees bounds, not lengths: few users alike whose bounds are far above them take four lists, too.  21 such calls,
// bounds of four times the longest: 1.000, from 0.983 to 1.014.  (Where the kernel looks at the
// lengths and chooses: the same.)
inline int list_spread(const Params& p, int64_t n_kt) {
    return (int64_t)p.batch * p.Hkv < 128 && n_kt >= 8 && (double)most_keys(p) > 2.5 * mean_keys(p) ? 2 : 0;
}

// key tiles of the longest user, NW x 32 history keys each
template <int NW>
int64_t list_tiles(const Params& p) {
    return ((int64_t)p.max_hist + NW * 32 - 1) / (NW * 32);
}

template <int D, int NW, bool TAILS, bool PW = false>
hipError_t launch_dkdv_as(const Params& p, hipStream_t s) {
    if (max_lead_keys(p) <= 0) return hipSuccess;
    const int64_t n_kt = list_tiles<NW>(p);
    const int spread = list_spread(p, n_kt);
    const int64_t n_items = work_grid((int64_t)p.batch * p.Hkv, n_kt, spread);
    const RowMap map = row_map(32, p.Hq, p.Hkv, max_query_rows(p));
    const int64_t resident = resident_workgroups<bwd_dkdv_kernel<D, NW, TAILS, PW>>(NW * 64);
    const int64_t persistent = n_items < resident ? n_items : resident;
    const int64_t tail_kt = p.rt_len ? (p.max_rt + 62) / 32 : 0;  // 32-key blocks behind the whole ones of the history
    const int64_t n_tails = p.rt_len ? work_grid((int64_t)p.batch * p.Hkv, tail_kt) : 0;
    if (n_items >= (1ll << 31) || persistent + n_tails >= (1ll << 31)) return hipErrorInvalidValue;
    Params pk = p;
    pk.queue = p.queue + QUEUE_DKDV * N_XCD;
    const int64_t n_blocks = persistent + (TAILS ? n_tails : 0);
    if (n_blocks > 0)
        hipLaunchKernelGGL((bwd_dkdv_kernel<D, NW, TAILS, PW>), dim3((unsigned)n_blocks), dim3(NW * 64), 0, s, pk, (int)n_kt, spread,
                           (unsigned)(n_items / N_XCD), (unsigned)persistent, map, (int)tail_kt);
    if constexpr (D == 128) {
        if (n_tails == 0) return hipGetLastError();
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((dkdv_tails_kernel<D, PW>), dim3((unsigned)n_tails), dim3(BRIEF_NW * 64), 0, s, p, map, (int)tail_kt);
    }
    return hipGetLastError();
}

// Users with few query rows against long histories (see bwd_dkdv_resident_kernel): do the host-known bounds allow it,
// and are there enough (user, kv head) items to give every compute unit one?  (A workgroup walks all keys of its item
// by itself: with fewer items the key tiles of the streaming kernel spread better.)  Whole backward passes of 92 such calls, 90 to 700 users of up to 2800
// keys: 0.92 of the time with the streaming kernel, eight of them slower by more than 3 %; those 15 that dkdv_brief_ways leaves here 0.87, none slower.
template <int D>
bool few_rows_per_user(const Params& p) {
    const int64_t max_units = ((max_query_rows(p) + 31) / 32) * (p.Hq / p.Hkv);
    return D == 64 && !p.rt_len && !p.pointwise && max_units > 0 && max_units <= DkdvResident<D, 12>::MAX_UNITS &&
           max_lead_keys(p) >= 512 && (int64_t)p.batch * p.Hkv >= 256;
}

template <int D>
hipError_t launch_dkdv_resident(const Params& p, hipStream_t s) {
    constexpr int NW = 12;
    const int64_t n_items = work_grid((int64_t)p.batch * p.Hkv, 1);
    if (n_items >= (1ll << 31)) return hipErrorInvalidValue;
    const int64_t resident = resident_workgroups<bwd_dkdv_resident_kernel<D, NW>>(NW * 64);
    Params pk = p;
    pk.queue = p.queue + QUEUE_DKDV * N_XCD;
    hipLaunchKernelGGL((bwd_dkdv_resident_kernel<D, NW>), dim3((unsigned)(n_items < resident ? n_items : resident)), dim3(NW * 64),
                       0, s, pk, (unsigned)(n_items / N_XCD));
    return hipGetLastError();
}

template <int D, int NW>
hipError_t launch_dkdv(const Params& p, hipStream_t s) {
    if constexpr (D == 64) {
        if (few_rows_per_user<D>(p)) return launch_dkdv_resident<D>(p, s);
    }
    if (p.pointwise) return p.rt_len ? launch_dkdv_as<D, NW, true, true>(p, s) : launch_dkdv_as<D, NW, false, true>(p, s);
    return p.rt_len ? launch_dkdv_as<D, NW, true>(p, s) : launch_dkdv_as<D, NW, false>(p, s);
}

}  // namespace
}  // namespace hta
