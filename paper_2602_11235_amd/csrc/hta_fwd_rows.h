// What the forward kernels share (hta_fwd_bf16.hip: batches that fill the chip; hta_serve_bf16.hip: a handful of
// requests): the row-stationary online softmax of one wave.
#pragma once
#include "hta_common.h"
#include "hta_rows.h"
#include "hta_tiles.h"

namespace hta {

constexpr float RESCALE_SLACK = 8.f;  // log2 units a row's logits may exceed its softmax reference before a rescale

// What a wave of the row-stationary forward pass keeps in registers -- the Q fragments of its RB blocks of 32 query
// rows (packed (row, head) pairs), the running softmax state and the O^T accumulators -- and the steps on it.
//
// RT: the users carry real-time tokens (mask rule 2).  Their keys follow the history keys in the K/V rows and run through
// the same tile loop; a sub-tile that reaches past the history is masked per query row with the row's limit
// (history + the real-time tokens strictly earlier than the row), and a real-time row gets its own key exactly like a target
// row.
//
// PW: the pointwise reading of phi2 -- weights norm * silu(scale s) on the same tiles and mask: no running maximum, no
// row sum, no lse; the accumulator holds sum_k s sigma(scale s) v and is scaled by norm * scale at the store.
template <int D, int RB, bool RT, bool PW>
struct FwdRows {
    static constexpr int NKS = D / 16, NDB = D / 32;
    bf16x8 qf[RB][NKS];  // B operand of S^T = K Q^T: lane = query row, 8 consecutive d values per k-step
    int lim[RB];         // leading keys the lane's row sees (RT; the history length otherwise)
    float m[RB], l[RB];
    floatx16 O[RB][NDB];
    // lane constants
    int nat[NKS], tlo[NDB], thi[NDB];  // element offsets of the operand fragments inside a swizzled tile
    int hf;
    float scale, c2, neg_c2;   // logits are handled in the log2 domain: c2 = scale log2(e)

    __device__ __forceinline__ void init_lane(const Params& p, int lane) {
        hf = lane >> 5;
        scale = p.scale;
        c2 = p.scale * LOG2E;
        neg_c2 = -c2;
        natural_offsets<D>(nat, lane);
        transposed_offsets<D>(tlo, thi, lane);
    }

    __device__ __forceinline__ void reset() {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            m[rb] = -INFINITY;
            l[rb] = 0.f;
#pragma unroll
            for (int db = 0; db < NDB; db++)
#pragma unroll
                for (int v = 0; v < 16; v++) O[rb][db][v] = 0.f;
        }
    }

    // Q fragments of the rows the lanes hold, and their limits
    __device__ __forceinline__ void load_q(const Params& p, const PackedRows& pr, int rho0, int64_t q_base, int L, int lane) {
        const int hf = lane >> 5;
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const PackedRows::Row x = pr.at(rho0 + rb * 32 + (lane & 31));
            const __bf16* qp = (const __bf16*)p.q + ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) qf[rb][ks] = *(const bf16x8*)(qp + ks * 16);
            lim[rb] = L;
        }
    }

    // Q fragments out of a swizzled tile of the wave's rows in LDS; L: the history length
    __device__ __forceinline__ void take_q(const __bf16* tile, int L) {
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
#pragma unroll
            for (int ks = 0; ks < NKS; ks++) qf[rb][ks] = *(const bf16x8*)(tile + rb * 32 * D + nat[ks]);
            lim[rb] = L;
        }
    }

    // Own key of target rows (rule 3) and of real-time rows, straight from global memory: where these rows' softmax starts
    // (reference = the own logit, weight 1), so the loads travel together with the Q fragments instead of in an
    // epilogue.  tok_shift: token index of query row 0.
    __device__ __forceinline__ void start_from_own_key(const Params& p, const PackedRows& pr, int rho0, int64_t kv_base, int g,
                                                       int tok_shift, int L, int lane) {
        const int hf = lane >> 5;
#pragma unroll
        for (int rb = 0; rb < RB; rb++) {
            const PackedRows::Row x = pr.at(rho0 + rb * 32 + (lane & 31));
            const int tok = tok_shift + x.row;
            if (tok >= L) {
                const int64_t off = ((kv_base + tok) * p.Hkv + g) * D;
                const __bf16* kp = (const __bf16*)p.k + off + 8 * hf;
                const __bf16* vp = (const __bf16*)p.v + off + 4 * hf;
                bf16x8 kk[NKS];
                bf16x4 vv[NDB][4];
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) kk[ks] = *(const bf16x8*)(kp + ks * 16);
#pragma unroll
                for (int db = 0; db < NDB; db++)
#pragma unroll
                    for (int v4 = 0; v4 < 4; v4++) vv[db][v4] = *(const bf16x4*)(vp + db * 32 + 8 * v4);
                float dot = 0.f;
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) dot = dot_bf16x8(dot, qf[rb][ks], kk[ks]);
                dot += other_half(dot);
                float ps = 1.f;
                if constexpr (PW) {
                    ps = pw_silu(dot, pw_sigmoid(dot, neg_c2));
                } else {
                    m[rb] = dot * c2;
                    l[rb] = hf == 0 ? 1.f : 0.f;
                }
#pragma unroll
                for (int db = 0; db < NDB; db++)
#pragma unroll
                    for (int v4 = 0; v4 < 4; v4++)
#pragma unroll
                        for (int j = 0; j < 4; j++) O[rb][db][4 * v4 + j] = ps * (float)vv[db][v4][j];
            }
        }
    }

    // One online-softmax step over a 32-key sub-tile that starts at key k0 (Ks, Vs: its first rows in LDS).  `n_live` =
    // number of keys of the sub-tile that exist (32 except in the ragged last tile), L = history length of the user.
    // TAIL: the sub-tile may be ragged or hold real-time keys.  Whole tiles of history keys, nearly all of a call, run an
    // instruction stream without the mask (215871 rows of 8/2 heads, 1.4 G pairs: with real-time tokens 519 -> 495 us,
    // pointwise 513 -> 503, softmax without real-time tokens the same 456).
    template <bool TAIL>
    __device__ __forceinline__ void subtile(const __bf16* Ks, const __bf16* Vs, int n_live, int k0, int L) {
        const bool masked = TAIL && RT && k0 + 32 > L;  // uniform: the sub-tile holds real-time keys (or runs past the end)
        if (masked) {
            bool any = false;
#pragma unroll
            for (int rb = 0; rb < RB; rb++) any = any || lim[rb] > k0;
            if (__builtin_amdgcn_ballot_w64(any) == 0) return;  // no row of this wave sees any key of the sub-tile
        }
        floatx16 S[1][RB];
        scores<1>(S, Ks);
        absorb<TAIL, 1>(S, Vs, n_live, k0, L);
    }

    // The two halves of a step over NS consecutive sub-tiles (NS = 2: one wave interleaves what two independent sub-tiles
    // wait for, where few waves share a SIMD).  S^T[key][row] = sum_d K[key][d] Q[row][d]
    template <int NS>
    __device__ __forceinline__ void scores(floatx16 (&S)[NS][RB], const __bf16* Ks) {
#pragma unroll
        for (int n = 0; n < NS; n++)
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int v = 0; v < 16; v++) S[n][rb][v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ks++)
#pragma unroll
            for (int n = 0; n < NS; n++) {
                const bf16x8 kf = *(const bf16x8*)(Ks + n * 32 * D + nat[ks]);
#pragma unroll
                for (int rb = 0; rb < RB; rb++) S[n][rb] = mfma32(kf, qf[rb][ks], S[n][rb]);
            }
    }

    // the same for one sub-tile with the Q fragments in LDS (`tile`: the wave's rows, swizzled), where registers do not hold them
    __device__ __forceinline__ void scores_of_lds(floatx16 (&S)[1][RB], const __bf16* Ks, const __bf16* tile) {
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            const bf16x8 kf = *(const bf16x8*)(Ks + nat[ks]);
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                S[0][rb] = mfma32(kf, *(const bf16x8*)(tile + rb * 32 * D + nat[ks]), ks == 0 ? zero : S[0][rb]);
            }
        }
    }

    // mask, weights and the PV products of the sub-tiles whose scores are S; first: no row has a reference (uniform)
    template <bool TAIL, int NS>
    __device__ __forceinline__ void absorb(floatx16 (&S)[NS][RB], const __bf16* Vs, int n_live, int k0, int L, bool first = false) {
        // Register v of the lane holds key 8 (v / 4) + 4 hf + v % 4 of the sub-tile; it is masked when that is >= the
        // number of visible keys, written as 4 hf - visible >= -(8 (v / 4) + v % 4): one subtraction per lane and
        // comparisons with constants, instead of sixteen lane constants kept in registers.
        if (TAIL && RT && k0 + 32 * NS > L) {  // per row: keys at or past the row's limit are not visible
            static_for<0, NS>([&](auto N) {
                static_for<0, RB>([&](auto Rb) {
                    constexpr int n = decltype(N)::value, rb = decltype(Rb)::value;
                    const int over = 4 * hf - (lim[rb] - k0 - 32 * n);
                    static_for<0, 16>([&](auto V) {
                        constexpr int v = decltype(V)::value;
                        S[n][rb][v] = (over >= -(8 * (v / 4) + (v % 4))) ? (PW ? PW_MASKED : -INFINITY) : S[n][rb][v];
                    });
                });
            });
        } else if (TAIL && n_live < 32 * NS) {  // ragged: keys >= L_b are not visible
#pragma unroll
            for (int n = 0; n < NS; n++) {
                const int over = 4 * hf - (n_live - 32 * n);
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    if (over >= -(8 * (v / 4) + (v % 4))) {
#pragma unroll
                        for (int rb = 0; rb < RB; rb++) S[n][rb][v] = PW ? PW_MASKED : -INFINITY;
                    }
                }
            }
        }
        bf16x8 pf[RB][2 * NS];
        if constexpr (PW) {
#pragma unroll
            for (int rb = 0; rb < RB; rb++)
#pragma unroll
                for (int v = 0; v < 16 * NS; v++)
                    pf[rb][v / 8][v % 8] = (__bf16)pw_silu(S[v / 16][rb][v % 16], pw_sigmoid(S[v / 16][rb][v % 16], neg_c2));  // s sigma(scale s): `scale` waits for the store
        } else {
            // Online softmax, one query row per lane (two lanes, 32 apart, share a row).  The reference m[rb]
            // of a row only has to bound its logits from above up to a modest factor: weights are exp2(s - m), sums
            // and outputs share the reference, and the final division by l removes it.  So the weights are formed
            // against the reference as it stands, without looking for the maximum first; the lane's sum of its 16
            // weights (per sub-tile) tells whether that was good enough: at most SUM_CAP = 16 * 2^RESCALE_SLACK when no logit exceeds
            // the reference by more than the slack (and inf or NaN while the reference is still -inf).  Only when some
            // lane of the wave fails that test -- in the first sub-tile of a row, and the handful of times a row
            // outgrows its reference -- is the maximum taken, the reference raised, the accumulators rescaled and
            // the weights formed again.  (The sum uses the rounded weights, the same as the P V product.)
            constexpr float SUM_CAP = 4096.f * NS;
            static_assert(RESCALE_SLACK == 8.f, "SUM_CAP is 16 * 2^RESCALE_SLACK");
            static_for<0, RB>([&](auto Rb) {
                constexpr int rb = decltype(Rb)::value;
                auto weights = [&](float ref) __attribute__((always_inline)) {
#pragma unroll
                    for (int v = 0; v < 16 * NS; v++)
                        pf[rb][v / 8][v % 8] = (__bf16)fast_exp2(fmaf(S[v / 16][rb][v % 16], c2, -ref));
                    float s0 = 0.f, s1 = 0.f;
#pragma unroll
                    for (int i = 0; i < 2 * NS; i++) add_bf16x8(s0, s1, pf[rb][i]);
                    return s0 + s1;
                };
                auto largest = [&]() __attribute__((always_inline)) {
                    float mx = S[0][rb][0];
#pragma unroll
                    for (int v = 1; v < 16 * NS; v++) mx = fmaxf(mx, S[v / 16][rb][v % 16]);
                    return fmaxf(mx, other_half(mx)) * c2;
                };
                // A caller that knows its first step (the request waves, whose key loop has few) takes the maximum at once instead
                // of failing the test: the same reference and bits.  The same tensors again and again, one 512 + 32 token request
                // 6.25 -> 5.76 us, 2048 + 128 8.59 -> 8.30, 8 of 512..4096 11.1 -> 10.5.  The ordinary kernel does not: its loop has 64 steps a user, and the branch's
                // registers cost more than one failure (training steps 0.997 .. 1.10 of the time).
                if (first) m[rb] = largest();
                // (a row that has seen no key yet has the reference -inf: with real-time masks it may hold only masked
                // logits; keep -inf - -inf out)
                float lt = weights(RT ? fmaxf(m[rb], -1e30f) : m[rb]);
                if (__builtin_amdgcn_ballot_w64(!(lt <= SUM_CAP)) != 0) {
                    const float mx = largest();
                    const bool grow = mx > m[rb] + RESCALE_SLACK;
                    const float m_new = grow ? mx : m[rb];
                    // 1 for the rows that keep their reference (which may still be -inf when rows see different keys)
                    const float alpha = grow ? fast_exp2(m[rb] - m_new) : 1.f;
                    m[rb] = m_new;
                    l[rb] *= alpha;
#pragma unroll
                    for (int db = 0; db < NDB; db++)
#pragma unroll
                        for (int v = 0; v < 16; v++) O[rb][db][v] *= alpha;
                    lt = weights(RT ? fmaxf(m_new, -1e30f) : m_new);
                }
                l[rb] += lt;
            });
        }
        // O^T[d][row] += sum_key V[key][d] P^T[key][row]
#pragma unroll
        for (int db = 0; db < NDB; db++)
#pragma unroll
            for (int s2 = 0; s2 < 2 * NS; s2++) {
                const bf16x8 vf = lds_read_tr_pair(Vs + 16 * s2 * D + tlo[db], Vs + 16 * s2 * D + thi[db]);
#pragma unroll
                for (int rb = 0; rb < RB; rb++) O[rb][db] = mfma32(vf, pf[rb][s2], O[rb][db]);
            }
    }
};

}  // namespace hta
