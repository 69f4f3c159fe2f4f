// dk/dv of the target tokens' own keys, for the launches of the backward pass that carry these blocks
// (hta_bwd_dq_bf16.hip, hta_bwd_brief_bf16.hip).
#pragma once
#include "hta_common.h"
#include "hta_mfma.h"

namespace hta {
namespace {

__device__ inline float group_sum(float x, int width) {  // sum over aligned groups of `width` lanes
    for (int o = width >> 1; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// ---------------------------------------------------------------------------------------- self keys
// One group of D/8 lanes per (target token, kv head); the group walks the r query heads of the kv head.  A block of
// THREADS threads takes the items block_x * IPB .. of user b.  HBM-bound and small (the target rows only); it has no
// launch of its own: its blocks are the last blocks of another grid, where they fill compute units that the tail of
// that one leaves idle.
// PW: pointwise weights, p = norm silu(x), ds = norm dp silu'(x) scale (no lse, no delta, `out` is not read).
template <int D, bool PW, int THREADS>
__device__ inline void bwd_self_block(const Params& p, int block_x, int b) {
    constexpr int LPR = D / 8;           // lanes per item, 8 elements (16 bytes) each
    constexpr int IPB = THREADS / LPR;   // items per block
    const int L = p.hist_len[b] + (p.rt_len ? p.rt_len[b] : 0), T = p.n_targets[b];  // L: tokens before the targets
    const int r = p.Hq / p.Hkv;
    const int item = block_x * IPB + threadIdx.x / LPR;  // (target, g) flattened, g fastest
    const int sub = threadIdx.x % LPR;
    const int t = item / p.Hkv, g = item % p.Hkv;
    if (t >= T) return;  // whole lane groups leave together; group_sum only talks inside a group
    const int64_t q_row = (int64_t)p.q_off[b] + (p.layer == 0 ? L + t : t);
    const __bf16* qg = (const __bf16*)p.q;
    const __bf16* dog = (const __bf16*)p.dout;
    const __bf16* og = (const __bf16*)p.out;
    const int64_t kv_off = (((int64_t)p.kv_off[b] + L + t) * p.Hkv + g) * D + sub * 8;
    const bf16x8 kk = *(const bf16x8*)((const __bf16*)p.k + kv_off);
    const bf16x8 vv = *(const bf16x8*)((const __bf16*)p.v + kv_off);
    float kself[8], vself[8], dk_t[8], dv_t[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
        kself[j] = (float)kk[j];
        vself[j] = (float)vv[j];
        dk_t[j] = 0.f;
        dv_t[j] = 0.f;
    }
    // N heads from h on, their loads together: four at a time instead of one keep enough in flight where targets are many (dQ launch and
    // the rest of a step at head_dim 128: 246 users of 28..115 + 31..127 targets 798 -> 784 us, 152 of 63..253 239 -> 234; without the own keys at
    // all 718 and 211).  At head_dim 32 the registers would cost the dQ kernel its fourth wave per SIMD (422 users 132 -> 137).
    auto heads = [&](int h, auto Count) __attribute__((always_inline)) {
        constexpr int N = decltype(Count)::value;
        bf16x8 qv[N], dov[N], ov[N];
        float lse[N];
#pragma unroll
        for (int i = 0; i < N; i++) {
            const int64_t off = (q_row * p.Hq + h + i) * D + sub * 8;
            qv[i] = *(const bf16x8*)(qg + off);
            dov[i] = *(const bf16x8*)(dog + off);
            if constexpr (!PW) {
                ov[i] = *(const bf16x8*)(og + off);
                lse[i] = p.lse[(int64_t)(h + i) * p.total_q + q_row];
            }
        }
#pragma unroll
        for (int i = 0; i < N; i++) {
            float dof[8], qf[8], part = 0.f, sp = 0.f, dpp = 0.f;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                dof[j] = (float)dov[i][j];
                qf[j] = (float)qv[i][j];
                if constexpr (!PW) part = fmaf(dof[j], (float)ov[i][j], part);
                sp = fmaf(qf[j], kself[j], sp);
                dpp = fmaf(dof[j], vself[j], dpp);
            }
            const float sc = group_sum(sp, LPR) * p.scale;
            const float dp = group_sum(dpp, LPR);
            float pw, ds;
            if constexpr (PW) {
                const float sg = 1.f / (1.f + __expf(-sc));
                pw = p.norm * pw_silu(sc, sg);
                ds = p.norm * dp * pw_silu_prime(sc, sg) * p.scale;
            } else {
                const float delta = group_sum(part, LPR);
                pw = __expf(sc - lse[i]);
                ds = pw * (dp - delta) * p.scale;
            }
#pragma unroll
            for (int j = 0; j < 8; j++) {
                dk_t[j] = fmaf(ds, qf[j], dk_t[j]);
                dv_t[j] = fmaf(pw, dof[j], dv_t[j]);
            }
        }
    };
    const int h_end = (g + 1) * r;
    int h = g * r;
    if constexpr (D > 32)
        for (; h + 4 <= h_end; h += 4) heads(h, std::integral_constant<int, 4>{});
    for (; h < h_end; h++) heads(h, std::integral_constant<int, 1>{});
    bf16x8 dk8, dv8;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        dk8[j] = (__bf16)dk_t[j];
        dv8[j] = (__bf16)dv_t[j];
    }
    *(bf16x8*)((__bf16*)p.dk + kv_off) = dk8;
    *(bf16x8*)((__bf16*)p.dv + kv_off) = dv8;
}

}  // namespace
}  // namespace hta
