// Entry points of the Python binding: the attention and normalization calls with their arguments in one packed block.
//
// ctypes converts every argument of a foreign call on its own (about 0.15 us each, 4 us for the 28 of an attention call,
// on top of launches of 2 us); the binding packs the arguments with one struct.pack instead and passes the address.
// Same checks, kernels, results and error codes as the functions of include/, which these forward to.  The block is
// read during the call and not kept.  The field order is that of the pack formats in hta.py and gln.py: pointers, then
// 8-byte, then 4-byte fields, nothing padded.
#include "../../include/mtfm_gln.h"
#include "../../include/mtfm_hta.h"
#include "../../include/mtfm_hta_pw.h"
#include "hta_common.h"

namespace {

enum Call { FWD = 0, BWD = 1, PW_FWD = 2, PW_BWD = 3 };

struct HtaArgs {
    const void *q, *k, *v;
    void* out;
    float* lse;
    const void* dout;
    void *dq, *dk, *dv;
    const int32_t *q_offsets, *kv_offsets, *hist_len, *n_targets, *rt_len, *timestamps;  // the last two null: no real-time tokens
    void* workspace;
    int64_t workspace_bytes, total_q, total_kv;
    int32_t batch, max_hist, max_rt, max_targets, Hq, Hkv, head_dim;
    float scale, norm;
    int32_t dtype, layer, call;
};
static_assert(sizeof(HtaArgs) == 16 * 8 + 3 * 8 + 12 * 4, "pack format 16P3q7i2f3i");

struct GlnArgs {
    const void *x, *gate;
    const int32_t* group_id;
    const float *gamma, *beta;
    void* y;
    float *mean, *rstd;
    const void* dy;
    void *dx, *dgate;
    float *dgamma, *dbeta;
    void* workspace;
    int64_t workspace_bytes, n_tokens, backward;
    int32_t d_model, n_groups;
    float eps;
    int32_t dtype;
};
static_assert(sizeof(GlnArgs) == 14 * 8 + 3 * 8 + 4 * 4, "pack format 14P3q2ifi");

// what the host knows of a bf16 call; false: no such call
bool sizes_of(const HtaArgs& a, hta::Params& p) {
    if (a.dtype != MTFM_HTA_BF16 || a.batch <= 0 || a.total_q <= 0) return false;
    p.batch = a.batch; p.total_q = a.total_q; p.total_kv = a.total_kv; p.max_hist = a.max_hist; p.max_targets = a.max_targets;
    p.Hq = a.Hq; p.Hkv = a.Hkv; p.d = a.head_dim == hta::BF16_PADDED_FROM ? hta::BF16_PADDED_TO : a.head_dim; p.layer = a.layer;
    if (a.rt_len && a.max_rt > 0) p.rt_len = a.rt_len, p.max_rt = a.max_rt;
    p.pointwise = a.call == PW_FWD || a.call == PW_BWD;
    return true;
}

}  // namespace

extern "C" {

MTFM_HTA_API int mtfm_binding_hta(const void* block, void* stream) {
    const HtaArgs& a = *(const HtaArgs*)block;
    const size_t ws = (size_t)a.workspace_bytes;
    switch (a.call) {
        case FWD:
            if (a.rt_len)
                return mtfm_hta_fwd_rt(a.q, a.k, a.v, a.out, a.lse, a.q_offsets, a.kv_offsets, a.hist_len, a.rt_len, a.n_targets,
                                       a.timestamps, a.batch, a.total_q, a.total_kv, a.max_hist, a.max_rt, a.max_targets, a.Hq,
                                       a.Hkv, a.head_dim, a.scale, a.dtype, a.layer, a.workspace, ws, stream);
            return mtfm_hta_fwd(a.q, a.k, a.v, a.out, a.lse, a.q_offsets, a.kv_offsets, a.hist_len, a.n_targets, a.batch,
                                a.total_q, a.total_kv, a.max_hist, a.max_targets, a.Hq, a.Hkv, a.head_dim, a.scale, a.dtype,
                                a.layer, a.workspace, ws, stream);
        case BWD:
            if (a.rt_len)
                return mtfm_hta_bwd_rt(a.dout, a.q, a.k, a.v, a.out, a.lse, a.dq, a.dk, a.dv, a.q_offsets, a.kv_offsets,
                                       a.hist_len, a.rt_len, a.n_targets, a.timestamps, a.batch, a.total_q, a.total_kv,
                                       a.max_hist, a.max_rt, a.max_targets, a.Hq, a.Hkv, a.head_dim, a.scale, a.dtype, a.layer,
                                       a.workspace, ws, stream);
            return mtfm_hta_bwd(a.dout, a.q, a.k, a.v, a.out, a.lse, a.dq, a.dk, a.dv, a.q_offsets, a.kv_offsets, a.hist_len,
                                a.n_targets, a.batch, a.total_q, a.total_kv, a.max_hist, a.max_targets, a.Hq, a.Hkv, a.head_dim,
                                a.scale, a.dtype, a.layer, a.workspace, ws, stream);
        case PW_FWD:
            if (a.rt_len)
                return mtfm_hta_pw_fwd_rt(a.q, a.k, a.v, a.out, a.q_offsets, a.kv_offsets, a.hist_len, a.rt_len, a.n_targets,
                                          a.timestamps, a.batch, a.total_q, a.total_kv, a.max_hist, a.max_rt, a.max_targets,
                                          a.Hq, a.Hkv, a.head_dim, a.scale, a.norm, a.dtype, a.layer, a.workspace, ws, stream);
            return mtfm_hta_pw_fwd(a.q, a.k, a.v, a.out, a.q_offsets, a.kv_offsets, a.hist_len, a.n_targets, a.batch, a.total_q,
                                   a.total_kv, a.max_hist, a.max_targets, a.Hq, a.Hkv, a.head_dim, a.scale, a.norm, a.dtype,
                                   a.layer, a.workspace, ws, stream);
        default:
            if (a.rt_len)
                return mtfm_hta_pw_bwd_rt(a.dout, a.q, a.k, a.v, a.dq, a.dk, a.dv, a.q_offsets, a.kv_offsets, a.hist_len,
                                          a.rt_len, a.n_targets, a.timestamps, a.batch, a.total_q, a.total_kv, a.max_hist,
                                          a.max_rt, a.max_targets, a.Hq, a.Hkv, a.head_dim, a.scale, a.norm, a.dtype, a.layer,
                                          a.workspace, ws, stream);
            return mtfm_hta_pw_bwd(a.dout, a.q, a.k, a.v, a.dq, a.dk, a.dv, a.q_offsets, a.kv_offsets, a.hist_len, a.n_targets,
                                   a.batch, a.total_q, a.total_kv, a.max_hist, a.max_targets, a.Hq, a.Hkv, a.head_dim, a.scale,
                                   a.norm, a.dtype, a.layer, a.workspace, ws, stream);
    }
}

// Which kernels the call of the block takes in bf16, by the rules that the library itself asks (all on sizes that the host knows; no pointer but
// rt_len, which is compared with null, is looked at).  For tests and measurements, which want to know what they run.
//   forward:  [0] pieces of keys (0: the ordinary kernel), [1] blocks of 32 rows per workgroup, [2] requests in a grid, not a list, [3] is there a
//             schedule's launch?
//   backward: [0] 0 two passes, 1 one pass, 2 brief; [1] waves that share a key block's rows (two passes: 0 for the kernels with a work queue),
//             [2] brief: dQ's workgroups in front; two passes with a queue: a user's rows resident; [3] is there a schedule's launch?
MTFM_HTA_API int mtfm_binding_hta_form(const void* block, int32_t* form) {
    const HtaArgs& a = *(const HtaArgs*)block;
    hta::Params p{};
    if (!sizes_of(a, p)) return MTFM_HTA_ERR_INVALID_ARG;
    if (a.call == FWD || a.call == PW_FWD) {
        p.n_splits = hta::serve_splits(p, hta::fwd_key_splits(p.batch, p.Hq, p.Hkv, p.d, hta::max_query_rows(p), hta::max_lead_keys(p)));
        form[0] = p.n_splits;
        form[1] = p.n_splits > 0 ? hta::serve_row_blocks(p) : hta::fwd_workgroup_rows(p) / 32;
        form[2] = p.n_splits > 0 && !hta::serve_takes_list(p);
        form[3] = p.n_splits == 0 && hta::forward_needs_schedule(p);
        return MTFM_HTA_OK;
    }
    const bool onepass = hta::bwd_is_onepass(p), brief = hta::bwd_is_brief(p);
    bool dq_first = false;
    form[0] = onepass ? 1 : brief ? 2 : 0;
    form[1] = onepass ? 0 : brief ? hta::bwd_brief_ways(p, &dq_first) : hta::dkdv_brief_ways(p);
    form[2] = brief ? dq_first : form[0] == 0 && form[1] == 0 && hta::dkdv_is_resident(p);
    form[3] = !brief && hta::backward_needs_schedule(p, onepass);
    return MTFM_HTA_OK;
}

// How a backward call of the block deals out its work, for tests: [0] one pass: is the next item taken late in the current one?  [1] two passes with a
// queue: the key tiles of a user go to 2^this lists.
MTFM_HTA_API int mtfm_binding_hta_lists(const void* block, int32_t* lists) {
    hta::Params p{};
    if (!sizes_of(*(const HtaArgs*)block, p)) return MTFM_HTA_ERR_INVALID_ARG;
    lists[0] = hta::onepass_asks_late(p);
    lists[1] = hta::dkdv_list_spread(p);
    return MTFM_HTA_OK;
}

MTFM_HTA_API int mtfm_binding_gln(const void* block, void* stream) {
    const GlnArgs& a = *(const GlnArgs*)block;
    if (!a.backward)
        return mtfm_gln_fwd(a.x, a.gate, a.group_id, a.gamma, a.beta, a.y, a.mean, a.rstd, a.n_tokens, a.d_model, a.n_groups,
                            a.eps, a.dtype, stream);
    return mtfm_gln_bwd(a.dy, a.x, a.gate, a.group_id, a.gamma, a.beta, a.mean, a.rstd, a.dx, a.dgate, a.dgamma, a.dbeta,
                        a.n_tokens, a.d_model, a.n_groups, a.dtype, a.workspace, (size_t)a.workspace_bytes, stream);
}

}  // extern "C"
