// bf16 forward kernel of Hybrid Target Attention for gfx950: QK^T and PV on the 32x32x16 bf16 MFMA
// with float32 accumulation, online softmax, K/V tiles staged in LDS once per key/value head and
// shared by the query heads of the GQA group (g = h / r, Section 3.2.2).
//
// Block skipping from the hybrid mask (rules 1 and 3): every query row of a user attends to all
// L_b history keys and never to another token's target key, so the only tiles ever issued are
// (row tile) x (history key tile); the single self key of a target row is where the row's online softmax starts.
// No mask is stored or loaded; only the ragged last history tile needs a bound check.
//
// Work decomposition: one workgroup = (user, kv head, tile of NW * 32 packed (row, head) pairs, see
// hta_rows.h), a wave = 32 of them, kept in registers.  S is computed transposed, S^T = K Q^T, so
// a lane owns one query row: the row maximum and sum are reductions over the lane's own
// registers plus one exchange with the other half of the wave, and P^T in accumulator layout is
// directly the B operand of O^T = V^T P^T.  V stays row-major in LDS and is read through the LDS
// transpose read.
//
// Batches of a few requests that leave most of the chip idle run hta_serve_bf16.hip instead.
#include "../../include/mtfm_hta.h"
#include "../../include/mtfm_hta_timing.h"
#include "hta_common.h"
#include "hta_fwd_rows.h"
#include "hta_mfma.h"
#include "hta_tiles.h"

namespace hta {
namespace {

constexpr int BN = 64;  // keys per LDS tile

// One workgroup per (user, kv head, chunk of query heads, row tile), from the launch grid.
template <int D, int NW, bool RT, bool PW = false>
__global__ __launch_bounds__(NW * 64, 2) void fwd_bf16_kernel(Params p, RowMap map, int spread) {
    using ST = KvStage<D, NW>;
    static_assert(ST::BN == BN, "tile height");
    // NSTAGE stages of [K tile][V tile], filled by asynchronous global -> LDS copies NSTAGE-1 tiles ahead of their use
    // (two ahead, except for d = 128 where a third stage would cost the second workgroup of the CU).  The compiler
    // never sees a store into this array (the copies are issued from inline assembly), so it neither orders LDS reads
    // against them nor drains them; the counted waits and barriers below do that.
    constexpr int NSTAGE = D <= 64 ? 3 : 2, AHEAD = NSTAGE - 1;
    // d = 128, two waves per SIMD: a tile's two sub-tiles as one step, so that a wave has two independent chains of products
    // and exponentials (11.6 -> 11.5 ms on 339 k rows of 16/2 heads, histories up to 8192); at d = 64 four waves do that.
    constexpr bool PAIRS = D == 128;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NSTAGE * ST::BYTES];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const WorkItem w = decode_spread(blockIdx.x, p.batch * p.Hkv * map.n_chunks, p.Hkv * map.n_chunks, map.n_tiles, spread);
    if (!w.valid) return;
    const int b = scheduled_user(p, w.user_slot);
    const int g = map.n_chunks == 1 ? w.y : w.y / map.n_chunks, chunk = w.y - g * map.n_chunks;
    const int L = p.hist_len[b], T = p.n_targets[b];
    const int LK = L + (RT ? p.rt_len[b] : 0);  // keys that run through the tile loop: history, then real-time
    const int n_rows = p.layer == 0 ? LK + T : T;
    if (w.tile * map.rows >= n_rows) return;  // uniform for the whole workgroup
    const PackedRows pr(map, w.tile, chunk, n_rows, g, p.Hq / p.Hkv);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int rho0 = wave_u * 32;
    const bool wave_live = pr.any_from(rho0);  // a wave behind the last row only helps staging
    const int tok_shift = p.layer == 0 ? 0 : LK;  // token index of query row 0
    const int64_t q_base = p.q_off[b], kv_base = p.kv_off[b];
    const __bf16* kg = (const __bf16*)p.k;
    const __bf16* vg = (const __bf16*)p.v;

    const int n_kt = (LK + BN - 1) / BN;
    uint32_t voff[ST::COPIES];
    ST::lane_offsets(voff, p.Hkv, wave, lane);
    const uint32_t smem_addr = lds_address(smem);

    // The first tiles are requested before the Q fragments: one memory latency instead of two
    // at the start of every workgroup.  From the wait on, the only vector-memory traffic of the loop are the
    // asynchronous copies, which this code counts itself; the compiler must not be left with pending loads of its own
    // (the Q fragments) that it would wait for inside the loop.
    if (n_kt > 0) ST::issue(kg, vg, kv_base, p.Hkv, g, LK, 0, smem_addr, voff, wave_u, lane);
    if (AHEAD > 1 && n_kt > 1) ST::issue(kg, vg, kv_base, p.Hkv, g, LK, 1, smem_addr + ST::BYTES, voff, wave_u, lane);
    FwdRows<D, 1, RT, PW> rows;
    rows.init_lane(p, lane);
    rows.load_q(p, pr, rho0, q_base, L, lane);
    if constexpr (RT) rows.lim[0] = p.lim[q_base + pr.at(rho0 + (lane & 31)).row];
    rows.reset();
    rows.start_from_own_key(p, pr, rho0, kv_base, g, tok_shift, L, lane);
    wait_vmem_loads();
    lds_barrier();
    // Tile t is consumed from stage t % NSTAGE while tile t+AHEAD is fetched
    // into stage (t+AHEAD) % NSTAGE, which was last read for tile t-1, i.e. before the barrier that every wave has passed.
    auto tile = [&](int t, auto St, auto Tail) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(Tail)::value;
        const int st = St;
        if (t + AHEAD < n_kt)
            ST::issue(kg, vg, kv_base, p.Hkv, g, LK, t + AHEAD, smem_addr + ((st + AHEAD) % NSTAGE) * ST::BYTES, voff, wave_u, lane);
        const __bf16* Ks = (const __bf16*)(smem + st * ST::BYTES);
        if (!wave_live) {
        } else if (PAIRS && !TAIL) {
            floatx16 S[2][1];
            rows.template scores<2>(S, Ks);
            rows.template absorb<false, 2>(S, Ks + ST::TILE, BN, t * BN, L);
        } else {
#pragma unroll
            for (int kb = 0; kb < BN / 32; kb++) {
                const int k0 = t * BN + kb * 32;
                if (!TAIL || k0 < LK)
                    rows.template subtile<TAIL>(Ks + kb * 32 * D, Ks + ST::TILE + kb * 32 * D, LK - k0, k0, L);
            }
        }
        // tile t+1 must have landed; a tile requested after it may stay in flight
        if (AHEAD > 1 && t + 2 < n_kt) wait_vmem_outstanding<ST::COPIES>(); else wait_vmem_outstanding<0>();
        lds_barrier();
    };
    // whole tiles of history keys first, then what needs a mask: at most one tile, more with real-time tokens
    const int n_whole = L / BN;
    for (int t = 0; t < n_whole; t += NSTAGE) {
        tile(t, std::integral_constant<int, 0>{}, std::false_type{});
        if (t + 1 < n_whole) tile(t + 1, std::integral_constant<int, 1>{}, std::false_type{});
        if constexpr (NSTAGE > 2) {
            if (t + 2 < n_whole) tile(t + 2, std::integral_constant<int, 2>{}, std::false_type{});
        }
    }
    for (int t = n_whole; t < n_kt; t++) tile(t, t % NSTAGE, std::true_type{});

    // normalisation and stores
    const int hf = lane >> 5;
    const PackedRows::Row x = pr.at(rho0 + (lane & 31));
    const float lt = rows.l[0] + other_half(rows.l[0]);
    if (!x.live) return;
    const float inv = PW ? p.norm * p.scale : 1.f / lt;
    __bf16* op = (__bf16*)p.out + ((q_base + x.row) * p.Hq + x.h) * D + 8 * hf;
    static_for<0, D / 16>([&](auto I) {
        constexpr int i = decltype(I)::value;
        *(bf16x8*)(op + 16 * i) = rows_of_16<i % 2>(rows.O[0][i / 2], inv);
    });
    if (!PW && hf == 0) p.lse[(int64_t)x.h * p.total_q + q_base + x.row] = (rows.m[0] + __builtin_amdgcn_logf(lt)) * LN2;
}

template <int D, int NW>
hipError_t launch(const Params& p, hipStream_t s) {
    void (*kernel)(Params, RowMap, int);
    if (p.pointwise)
        kernel = p.rt_len ? fwd_bf16_kernel<D, NW, true, true> : fwd_bf16_kernel<D, NW, false, true>;
    else
        kernel = p.rt_len ? fwd_bf16_kernel<D, NW, true> : fwd_bf16_kernel<D, NW, false>;
    const int64_t rows = max_query_rows(p);
    if (rows <= 0) return hipSuccess;
    const RowMap map = row_map(NW * 32, p.Hq, p.Hkv, rows);
    const int64_t groups = (int64_t)p.batch * p.Hkv * map.n_chunks;
    const int spread = grid_spread(p, groups, map.n_tiles);
    const int64_t n_blocks = work_grid(groups, map.n_tiles, spread);
    if (n_blocks >= (1ll << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel, dim3((unsigned)n_blocks), dim3(NW * 64), 0, s, p, map, spread);
    return hipGetLastError();
}

// Waves per workgroup, one 32-row block each (two per wave, sharing the operand reads, were slower at every head shape once rows
// came packed: 340 against 308 us on 338 users at 4/4 heads).  At head_dim 64 eight waves, two workgroups per unit, share each
// K/V tile among 256 rows; four waves where 256 rows are too coarse for the users: few rows in a full layer (8/2 heads, P
// packed rows per user: P = 480 44 against 68 us, P = 1400 37 against 36, P = 3400 470 against 450), or just more than 256
// at most (P = 92..372: 88 against 115 us).  At 128 (1.05 against 1.13 ms on 232 users of 252..1010 keys, 46 -> 39 us on 44 short
// ones) and 32 four waves always.
int waves(const Params& p) {
    if (p.d != 64) return 4;
    const int64_t r = p.Hq / p.Hkv, most = max_query_rows(p) * r;
    const bool four = p.layer == 0 ? mean_rows(p) * r <= 1000. && most > 256 : most > 256 && most <= 384;
    return four ? 4 : 8;
}

}  // namespace

bool bf16_supported(int32_t d, int32_t Hq, int32_t Hkv) {
    (void)Hq;
    (void)Hkv;
    return d == 32 || d == 64 || d == 128;
}

int fwd_workgroup_rows(const Params& p) { return waves(p) * 32; }

hipError_t launch_fwd_bf16(const Params& p, hipStream_t s) {
    if (p.n_splits > 0) return launch_serve_bf16(p, s);
    hipError_t e;
    timing_begin(MTFM_HTA_KERNEL_FWD, s);
    switch (p.d) {
        case 32: e = launch<32, 4>(p, s); break;
        case 64: e = waves(p) == 4 ? launch<64, 4>(p, s) : launch<64, 8>(p, s); break;
        case 128: e = launch<128, 4>(p, s); break;
        default: e = hipErrorInvalidValue;
    }
    timing_end(MTFM_HTA_KERNEL_FWD, s);
    return e;
}

}  // namespace hta
