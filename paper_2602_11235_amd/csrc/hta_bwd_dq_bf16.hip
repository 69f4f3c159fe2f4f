// bf16 backward of Hybrid Target Attention for gfx950, first launch: dQ (and the self-key blocks).
//
// Gradient of A = softmax_visible(scale Q K^T) V (the two attention equations of Section 3.2.2)
// with the probabilities recomputed from the saved logsumexp:
//   P = exp(scale S - lse),  dP = dO V^T,  dS = P o (dP - delta),  delta_i = <dO_i, O_i>,  dQ = scale dS K
// The whole backward pass is three pieces of work in two launches (see hta_bwd_bf16.hip); this file holds
//   1. bwd_self: the self-key terms of target rows' keys (rule 3: a target key is seen by its own row
//      only, so its dk/dv come from that row alone and are written here, final, in bf16).  Its blocks
//      are the last blocks of the dQ grid.
//   2. bwd_dq:   row-stationary, the forward kernel's decomposition: a wave keeps query rows (Q, dO, dQ) in
//      registers and streams the history K/V tiles through LDS.  S^T = K Q^T and dP^T = V dO^T have
//      the query row on the lane, so lse and delta are one register each and dS^T in accumulator layout
//      is directly the k-operand of dQ^T = K^T dS^T.  The self key of a target row is where its dQ
//      starts.  dq is written once.  delta_i = <dO_i, O_i> is formed here, from the dO fragments
//      the wave holds anyway, and left (negated, with -lse/scale) in the workspace for the dK/dV launch.
// A translation unit of its own because it is compiled with another instruction scheduling strategy than the rest of
// the library (build.py: the strategy that favours instruction-level parallelism interleaves matrix products
// with weight arithmetic, which the default, occupancy-driven strategy does not).
#include "../../include/mtfm_hta.h"
#include "hta_bwd_self.h"
#include "hta_common.h"
#include "hta_mfma.h"
#include "hta_rows.h"
#include "hta_tiles.h"

namespace hta {
namespace {

// ---------------------------------------------------------------------------------------- dQ
constexpr int BN = 64;  // keys per LDS tile of the dQ kernel

// RT: users with real-time tokens (mask rule 2), handled as in the forward kernel: their keys run through the same
// tile loop, masked per query row with the row's limit; a real-time row's dQ starts from its own key.
// PW: the pointwise reading of phi2 -- dS = dP o silu'(scale S), scaled by norm * scale at the store; no lse, no
// delta, `out` is not read.  The row statistics the dK/dV pass starts its accumulators from are left as zeros.
// Blocks n_dq .. of the grid are the self-key blocks (bwd_self_block), self_bpu per user.
template <int D, int RB, int NW, bool RT, bool PW = false>
__global__ __launch_bounds__(NW * 64, D == 64 && RB == 1 && NW == 4 ? 3 : 2) void bwd_dq_kernel(Params p, RowMap map, int spread, unsigned n_dq,
                                                                                            unsigned self_bpu) {
    if (blockIdx.x >= n_dq) {  // uniform for the block, and before any barrier
        const unsigned sb = blockIdx.x - n_dq;
        bwd_self_block<D, PW, NW * 64>(p, (int)(sb % self_bpu), (int)(sb / self_bpu));
        return;
    }
    using ST = KvStage<D, NW>;
    constexpr int NKS = D / 16, NDB = D / 32, NKB = BN / 32;
    static_assert(ST::BN == BN, "tile height");
    // NSTAGE stages of [K tile][V tile], filled by asynchronous global -> LDS copies NSTAGE-1 tiles ahead of their use
    // (two ahead, except for d = 128 where a third stage would cost the second workgroup of the CU).  The compiler
    // never sees a store into this array (the copies are issued from inline assembly), so it neither orders LDS reads
    // against them nor drains them; the counted waits and barriers below do that.
    constexpr int NSTAGE = D <= 64 ? 3 : 2, AHEAD = NSTAGE - 1;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NSTAGE * ST::BYTES];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
    // behind the -lse/scale array: what the S accumulators of rows that do not exist start from in the dK/dV pass
    if (blockIdx.x == 0 && tid == 0) p.neg_lse_s[(int64_t)p.Hq * p.total_q] = -1e30f;
    const WorkItem w = decode_spread(blockIdx.x, p.batch * p.Hkv * map.n_chunks, p.Hkv * map.n_chunks, map.n_tiles, spread);
    if (!w.valid) return;
    const int b = scheduled_user(p, w.user_slot);
    const int g = map.n_chunks == 1 ? w.y : w.y / map.n_chunks, chunk = w.y - g * map.n_chunks;
    const int L = p.hist_len[b], T = p.n_targets[b];
    const int LK = L + (RT ? p.rt_len[b] : 0);  // keys that run through the tile loop: history, then real-time
    const int n_rows = p.layer == 0 ? LK + T : T;
    if (w.tile * map.rows >= n_rows) return;  // uniform for the whole workgroup
    const PackedRows pr(map, w.tile, chunk, n_rows, g, p.Hq / p.Hkv);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave), rho0 = wave_u * RB * 32;
    const bool wave_live = pr.any_from(rho0);  // a wave behind the last row only helps staging
    const int tok_shift = p.layer == 0 ? 0 : LK;
    const int64_t q_base = p.q_off[b], kv_base = p.kv_off[b];
    const __bf16* kg = (const __bf16*)p.k;
    const __bf16* vg = (const __bf16*)p.v;
    const float c2 = p.scale * LOG2E;
    const float neg_c2 = -c2;

    const int n_kt = (LK + BN - 1) / BN;
    int nat[NKS], tlo[NDB], thi[NDB];  // per-lane element offsets of the operand fragments inside a swizzled tile
    natural_offsets<D>(nat, lane);
    transposed_offsets<D>(tlo, thi, lane);
    uint32_t voff[ST::COPIES];
    ST::lane_offsets(voff, p.Hkv, wave, lane);
    const uint32_t smem_addr = lds_address(smem);

    // the first K/V tiles are requested before the row operands are loaded and delta is formed: their latencies overlap
    if (n_kt > 0) ST::issue(kg, vg, kv_base, p.Hkv, g, LK, 0, smem_addr, voff, wave_u, lane);
    if (AHEAD > 1 && n_kt > 1) ST::issue(kg, vg, kv_base, p.Hkv, g, LK, 1, smem_addr + ST::BYTES, voff, wave_u, lane);

    // per lane: one query row per row block (clamped past the end; never stored then)
    bf16x8 qf[RB][NKS], dof[RB][NKS];
    float lse2[RB], dl[RB];
    int lim[RB];  // RT: leading keys the lane's row sees
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
        const PackedRows::Row x = pr.at(rho0 + rb * 32 + l32);
        const int64_t off = ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
        float part = 0.f;  // this lane's half of delta = <dO, O>
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            qf[rb][ks] = *(const bf16x8*)((const __bf16*)p.q + off + ks * 16);
            dof[rb][ks] = *(const bf16x8*)((const __bf16*)p.dout + off + ks * 16);
            if constexpr (!PW) part = dot_bf16x8(part, dof[rb][ks], *(const bf16x8*)((const __bf16*)p.out + off + ks * 16));
        }
        const int64_t stat = (int64_t)x.h * p.total_q + q_base + x.row;
        const float lse = PW ? 0.f : p.lse[stat];
        const float delta = part + other_half(part);
        lse2[rb] = lse * LOG2E;
        dl[rb] = -delta;
        lim[rb] = RT ? p.lim[q_base + x.row] : L;
        // every (row, head) belongs to exactly one wave of this kernel: it leaves the row statistics for the dK/dV pass
        if (x.live && hf == 0) {
            p.neg_delta[stat] = -delta;
            p.neg_lse_s[stat] = -lse / p.scale;
        }
    }
    floatx16 dQ[RB][NDB];  // dQ^T: [d (registers)][row (lanes)]
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int v = 0; v < 16; v++) dQ[rb][db][v] = 0.f;
        // the own key of target rows (rule 3) and of real-time rows: where their dQ starts
        const int tok = tok_shift + pr.at(rho0 + rb * 32 + l32).row;
        if (tok >= L) {
            const int64_t off = ((kv_base + tok) * p.Hkv + g) * D;
            bf16x8 kk[NKS], vv[NKS];
            bf16x4 kt[NDB][4];
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) {
                kk[ks] = *(const bf16x8*)(kg + off + ks * 16 + 8 * hf);
                vv[ks] = *(const bf16x8*)(vg + off + ks * 16 + 8 * hf);
            }
#pragma unroll
            for (int db = 0; db < NDB; db++)
#pragma unroll
                for (int v4 = 0; v4 < 4; v4++) kt[db][v4] = *(const bf16x4*)(kg + off + db * 32 + 8 * v4 + 4 * hf);
            float sp = 0.f, dpp = 0.f;
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) {
                sp = dot_bf16x8(sp, qf[rb][ks], kk[ks]);
                dpp = dot_bf16x8(dpp, dof[rb][ks], vv[ks]);
            }
            sp += other_half(sp);
            dpp += other_half(dpp);
            float ds;
            if constexpr (PW) ds = dpp * pw_silu_prime(sp * p.scale, pw_sigmoid(sp, neg_c2));
            else ds = fast_exp2(fmaf(sp, c2, -lse2[rb])) * (dpp + dl[rb]);
#pragma unroll
            for (int db = 0; db < NDB; db++)
#pragma unroll
                for (int v4 = 0; v4 < 4; v4++)
#pragma unroll
                    for (int j = 0; j < 4; j++) dQ[rb][db][4 * v4 + j] = ds * (float)kt[db][v4][j];
        }
    }

    // The dP products start from -delta instead of zero.  With one row block per wave sixteen registers are free to keep it in (opaque,
    // or they would be written anew for every sub-tile), which takes sixteen additions of about seventy vector instructions out of a
    // sub-tile: head_dim 64 with real-time tokens 0.691 -> 0.676 ms (256 users of 512..1024 keys), head_dim 128 16.6 -> 16.2 ms
    // (128 users of 750..8192 keys).  With two row blocks thirteen registers for the copies of a last, ragged tile then wait in scratch, 0.2 GB
    // of traffic on 256 users of 512..1024 keys, and it pays on longer ones only: whole steps with the additions instead, in turn on one
    // box, 1807 against 1804 us there (another draw of the lengths 1787 against 1792), 2669 against 2658 on 256 users of 1024
    // keys, 4680 against 4641 on 83 users of 461..4062.
    floatx16 dp0[RB];
    if constexpr (!PW) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
#pragma unroll
            for (int v = 0; v < 16; v++) dp0[rb][v] = dl[rb];
            if constexpr (RB == 1) asm volatile("" : "+v"(dp0[rb]));
        }
    }

    auto subtile = [&](const __bf16* Ks, const __bf16* Vs, int n_live, int k0) __attribute__((always_inline)) {  // Ks, Vs: first row of the sub-tile (key k0)
        const bool masked = RT && k0 + 32 > L;  // uniform: the sub-tile holds real-time keys (or runs past the end)
        if (masked) {
            bool any = false;
#pragma unroll
            for (int rb = 0; rb < RB; rb++) any = any || lim[rb] > k0;
            if (__builtin_amdgcn_ballot_w64(any) == 0) return;  // no row of this wave sees any key of the sub-tile
        }
        floatx16 S[RB], dP[RB];  // S^T, dP^T: [key (registers)][row (lanes)]
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            const bf16x8 kf = *(const bf16x8*)(Ks + nat[ks]);
            const bf16x8 vf = *(const bf16x8*)(Vs + nat[ks]);
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                if (ks == 0) {
                    const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    S[rb] = mfma32(kf, qf[rb][ks], zero);
                    dP[rb] = mfma32(vf, dof[rb][ks], PW ? zero : dp0[rb]);
                } else {
                    S[rb] = mfma32(kf, qf[rb][ks], S[rb]);
                    dP[rb] = mfma32(vf, dof[rb][ks], dP[rb]);
                }
            }
        }
        // Register v of the lane holds key 8 (v / 4) + 4 hf + v % 4 of the sub-tile; it is masked when that is >= the
        // number of visible keys, written as 4 hf - visible >= -(8 (v / 4) + v % 4): one subtraction per lane and
        // comparisons with constants, instead of sixteen lane constants kept in registers.
        if (masked) {  // per row: keys at or past the row's limit are not visible (P = 0)
            static_for<0, RB>([&](auto Rb) {
                constexpr int rb = decltype(Rb)::value;
                const int over = 4 * hf - (lim[rb] - k0);
                static_for<0, 16>([&](auto V) {
                    constexpr int v = decltype(V)::value;
                    S[rb][v] = (over >= -(8 * (v / 4) + (v % 4))) ? (PW ? PW_MASKED : -INFINITY) : S[rb][v];
                });
            });
        } else if (n_live < 32) {  // ragged: keys >= L_b are not visible (P = 0)
            const int over = 4 * hf - n_live;
#pragma unroll
            for (int v = 0; v < 16; v++) {
                if (over >= -(8 * (v / 4) + (v % 4))) {
#pragma unroll
                    for (int rb = 0; rb < RB; rb++) S[rb][v] = PW ? PW_MASKED : -INFINITY;
                }
            }
        }
        bf16x8 dsb[RB][2];
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int v = 0; v < 16; v++) {
                if constexpr (PW) {
                    const float sg = pw_sigmoid(S[rb][v], neg_c2);
                    dsb[rb][v / 8][v % 8] = (__bf16)(dP[rb][v] * pw_silu_prime_of_logit(S[rb][v], sg, p.scale));
                } else {
                    const float pw = fast_exp2(fmaf(S[rb][v], c2, -lse2[rb]));
                    dsb[rb][v / 8][v % 8] = (__bf16)(pw * dP[rb][v]);
                }
            }
        // dQ^T[d][row] += sum_key K[key][d] dS^T[key][row]
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2; s2++) {
                const bf16x8 ktf = lds_read_tr_pair(Ks + 16 * s2 * D + tlo[db], Ks + 16 * s2 * D + thi[db]);
#pragma unroll
                for (int rb = 0; rb < RB; rb++) dQ[rb][db] = mfma32(ktf, dsb[rb][s2], dQ[rb][db]);
            }
    };

    // From here on the only vector-memory traffic of the loop are the asynchronous copies, which this code counts
    // itself; the compiler must not be left with pending loads of its own (Q, dO, O, lse) that it would wait for
    // inside the loop.  (The first tiles were requested before those loads.)
    wait_vmem_loads();
    lds_barrier();
    // Tile t is consumed from stage t % NSTAGE while tile t+AHEAD is fetched into stage (t+AHEAD) % NSTAGE, which was
    // last read for tile t-1, i.e. before the barrier that every wave has passed.
    auto tile = [&](int t, auto St) __attribute__((always_inline)) {
        constexpr int st = decltype(St)::value;
        if (t + AHEAD < n_kt)
            ST::issue(kg, vg, kv_base, p.Hkv, g, LK, t + AHEAD, smem_addr + ((st + AHEAD) % NSTAGE) * ST::BYTES, voff, wave_u, lane);
        const __bf16* Ks = (const __bf16*)(smem + st * ST::BYTES);
        const __bf16* Vs = Ks + ST::TILE;
        const int live = LK - t * BN;  // keys of this tile that exist (>= 1)
#pragma unroll
        for (int kb = 0; kb < NKB; kb++) {
            const int n_live = live - kb * 32;
            if (wave_live && n_live > 0) subtile(Ks + kb * 32 * D, Vs + kb * 32 * D, n_live, t * BN + kb * 32);
        }
        // tile t+1 must have landed; a tile requested after it may stay in flight
        if (AHEAD > 1 && t + 2 < n_kt) wait_vmem_outstanding<ST::COPIES>(); else wait_vmem_outstanding<0>();
        lds_barrier();
    };
    for (int t = 0; t < n_kt; t += NSTAGE) {
        tile(t, std::integral_constant<int, 0>{});
        if (t + 1 < n_kt) tile(t + 1, std::integral_constant<int, 1>{});
        if constexpr (NSTAGE > 2) {
            if (t + 2 < n_kt) tile(t + 2, std::integral_constant<int, 2>{});
        }
    }

    __bf16* dqg = (__bf16*)p.dq;
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
        const PackedRows::Row x = pr.at(rho0 + rb * 32 + l32);
        if (x.live) {
            __bf16* op = dqg + ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
            static_for<0, D / 16>([&](auto I) {
                constexpr int i = decltype(I)::value;
                *(bf16x8*)(op + 16 * i) = rows_of_16<i % 2>(dQ[rb][i / 2], PW ? p.scale * p.norm : p.scale);
            });
        }
    }
}

template <int D, int RB, int NW>
hipError_t launch_dq(const Params& p, hipStream_t s) {
    const int64_t rows = max_query_rows(p);
    if (rows <= 0) return hipSuccess;
    const RowMap map = row_map(NW * RB * 32, p.Hq, p.Hkv, rows);
    const int64_t groups = (int64_t)p.batch * p.Hkv * map.n_chunks;
    const int spread = grid_spread(p, groups, map.n_tiles);
    const int64_t n_blocks = work_grid(groups, map.n_tiles, spread);
    // the self-key blocks: (target, kv head) items of every user, NW * 64 / (D / 8) per block
    constexpr int IPB = NW * 64 / (D / 8);
    const int64_t self_bpu = ((int64_t)p.max_targets * p.Hkv + IPB - 1) / IPB;
    const int64_t n_self = self_bpu * p.batch;
    if (n_blocks + n_self >= (1ll << 31)) return hipErrorInvalidValue;
    auto kernel = bwd_dq_kernel<D, RB, NW, false>;
    if constexpr (RB == 1) {
        if (p.pointwise) kernel = p.rt_len ? bwd_dq_kernel<D, RB, NW, true, true> : bwd_dq_kernel<D, RB, NW, false, true>;
        else if (p.rt_len) kernel = bwd_dq_kernel<D, RB, NW, true>;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_blocks + n_self)), dim3(NW * 64), 0, s, p, map, spread, (unsigned)n_blocks,
                       (unsigned)(self_bpu > 0 ? self_bpu : 1));
    return hipGetLastError();
}

}  // namespace

// Four waves per workgroup.  At head_dim 64 one row block per wave and three workgroups per unit (158 registers): finer than two
// blocks per wave and two workgroups, and faster wherever that counts (P packed rows per user: P = 92..372 189 -> 114 us,
// P = 790 469 -> 366, P = 1400 52 -> 46, P = 3400 612 -> 600).  Two blocks per wave share the operand reads, which draws less power and shows once a call runs for
// long: 83 users of 461..4062 keys 954 -> 909 us, and a whole step of 256 users of 512..1024 keys 1819 -> 1801.  At 128 four
// waves, two workgroups per unit, instead of eight: 1.68 -> 1.56 ms on 232 users of 252..1010 keys, 66 -> 52 us on 44 short ones.
hipError_t launch_bwd_dq_bf16(const Params& p, hipStream_t s) {
    const double packed = mean_rows(p) * (p.Hq / p.Hkv);
    const bool two_blocks = packed >= 2000. && packed * p.batch * p.Hkv >= 2000. * 256. && !p.rt_len && !p.pointwise;
    switch (p.d) {
        case 32: return launch_dq<32, 1, 4>(p, s);
        case 64: return two_blocks ? launch_dq<64, 2, 4>(p, s) : launch_dq<64, 1, 4>(p, s);
        default: return launch_dq<128, 1, 4>(p, s);
    }
}

}  // namespace hta
