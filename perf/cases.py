"""Workloads the library is timed on: what a ranking model asks of it in training and in serving.

A case is a dict of plain values.  `listed()` names a dozen, `draw(rng)` gives others of the same ranges, `prepare` puts
a program's state on the GPU (inputs, buffers, lengths), `run` is one pass over it through the public entry points, `work`
the bytes and operations of a pass that no implementation can do without, `tolerance` how far two correct
implementations of the same precision may lie apart.

The jagged lengths, and with real-time tokens the timestamps, are part of a case (drawn from its `lengths_seed`), the
tensors' values come from the seed given to `prepare`.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_11235_amd import gln, hta, hta_pw, inputs

# head shapes in use: (query heads, key/value heads, head_dim)
HEADS = ((8, 2, 64), (16, 4, 64), (16, 2, 128), (4, 2, 32), (4, 4, 64))


def _attention(name, op, layer, batch, hist, targets, heads, seed, rt=(0, 0), reading="softmax", hist_kind="uniform",
               std=0.3):
    """op: "infer" (forward only) or "train" (forward, then backward).  hist_kind "uniform": history lengths uniform in
    [hist_lo, hist_hi]; "pareto": hist_lo / u capped at hist_hi, u uniform in (0, 1): a heavy tail of long histories."""
    case = dict(op=op, reading=reading, layer=layer, batch=batch, hist_kind=hist_kind, hist_lo=hist[0], hist_hi=hist[1],
                tgt_lo=targets[0], tgt_hi=targets[1], rt_lo=rt[0], rt_hi=rt[1], Hq=heads[0], Hkv=heads[1],
                head_dim=heads[2], std=std, lengths_seed=seed)
    if name:
        case["name"] = name
    return case


def _gln(name, op, tokens, d_model, groups, gated):
    """op: "gln_infer" (forward, no statistics kept) or "gln_train" (forward, then backward)."""
    case = dict(op=op, tokens=tokens, d_model=d_model, groups=groups, gated=gated)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # Serving, one request: a user's history and the candidates of one scenario.  The smallest attention call.
        _attention("serve_one", "infer", "target", 1, (2048, 2048), (128, 128), (8, 2, 64), 21),
        # Serving, a few requests of unlike lengths scored in one call.
        _attention("serve_batch", "infer", "target", 8, (512, 4096), (16, 128), (8, 2, 64), 22),
        # Serving, very long histories and wide heads.
        _attention("serve_long", "infer", "target", 4, (8192, 8192), (64, 64), (16, 2, 128), 23),
        # Serving with the user's real-time behaviour (visible only to later tokens).
        _attention("serve_realtime", "infer", "target", 8, (512, 4096), (16, 128), (8, 2, 64), 24, rt=(16, 96)),
        # Training step of a full layer on a small batch of short histories.
        _attention("train_short", "train", "full", 64, (128, 512), (32, 32), (8, 2, 64), 1),
        # Training step of a full layer: the workload of the headline figure.
        _attention("train_full", "train", "full", 256, (512, 1024), (64, 64), (8, 2, 64), 2),
        # The same with real-time tokens.
        _attention("train_realtime", "train", "full", 256, (512, 1024), (64, 64), (8, 2, 64), 12, rt=(32, 128)),
        # Training step of a target-only layer: few query rows per user against long shared histories.
        _attention("train_target", "train", "target", 512, (2048, 2048), (128, 128), (16, 4, 64), 3),
        # Training step over heavy-tailed histories with wide heads.  The largest call.
        _attention("train_long", "train", "full", 128, (750, 8192), (16, 256), (16, 2, 128), 4, hist_kind="pareto"),
        # Training step with pointwise (SiLU) attention weights instead of a softmax.
        _attention("train_pointwise", "train", "full", 256, (512, 1024), (64, 64), (8, 2, 64), 2, reading="pointwise"),
        # Group layer normalization in training: gated, every token of the headline batch.
        _gln("norm_train", "gln_train", 215871, 512, 8, True),
        # Group layer normalization in serving: the tokens of one request.
        _gln("norm_serve", "gln_infer", 2176, 512, 8, False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("serve", "train", "long", "norm"), (4, 5, 1, 2))[0]
    seed = rng.randrange(1 << 20)
    if kind == "norm":
        d_model = 8 * rng.randint(16, 128)
        groups = rng.randint(1, 8)
        op = rng.choice(("gln_infer", "gln_train"))
        tokens = _log_int(rng, 64, 8192) if op == "gln_infer" else _log_int(rng, 2048, 262144)
        return _gln(None, op, tokens, d_model, groups, rng.random() < 0.6)
    if kind == "serve":
        hi = _log_int(rng, 256, 8192)
        lo = hi if rng.random() < 0.3 else max(1, hi // 8)
        t_hi = _log_int(rng, 8, 256)
        rt = (8, rng.randint(16, 128)) if rng.random() < 0.3 else (0, 0)
        return _attention(None, "infer", "target", _log_int(rng, 1, 32), (lo, hi), (max(1, t_hi // 8), t_hi),
                          rng.choice(HEADS[:3]), seed, rt=rt, std=rng.choice((0.3, 0.6, 1.0)))
    if kind == "long":
        return _attention(None, "train", "full", _log_int(rng, 16, 96), (rng.randint(300, 750), _log_int(rng, 2048, 8192)),
                          (16, rng.randint(32, 256)), rng.choice(((16, 2, 128), (8, 2, 64))), seed, hist_kind="pareto")
    layer = rng.choice(("full", "full", "target"))
    hi = _log_int(rng, 96, 2048)
    t_hi = rng.randint(8, 128)
    # (a batch of full layers is bounded by its pairs: 512 short histories or a few dozen long ones)
    batch = _log_int(rng, 16, max(32, min(512, int(6e8 / (hi * hi)))) if layer == "full" else 512)
    rt = (8, rng.randint(16, 128)) if rng.random() < 0.25 else (0, 0)
    return _attention(None, "train", layer, batch, (max(1, hi // rng.choice((1, 2, 4))), hi), (max(1, t_hi // 4), t_hi),
                      rng.choices(HEADS, (4, 2, 2, 1, 1))[0], seed, rt=rt,
                      reading="pointwise" if rng.random() < 0.2 else "softmax", std=rng.choice((0.3, 0.6, 1.0)))


# ------------------------------------------------------------------------------------------------- lengths of a case
def _uniform_ints(seed, stream, n, lo, hi):
    u = inputs.uniform01(inputs.stream_key(seed, stream), 0, n)
    return np.minimum(hi, lo + np.floor(u * (hi - lo + 1)).astype(np.int64)).astype(np.int32)


def _lengths(case):
    seed, n = case["lengths_seed"], case["batch"]
    if case["hist_kind"] == "pareto":
        u = inputs.uniform01(inputs.stream_key(seed, 0), 0, n)
        hist = np.minimum(case["hist_hi"], np.floor(case["hist_lo"] / u)).astype(np.int32)
    else:
        hist = _uniform_ints(seed, 0, n, case["hist_lo"], case["hist_hi"])
    tgt = _uniform_ints(seed, 1, n, case["tgt_lo"], case["tgt_hi"])
    rt = _uniform_ints(seed, 6, n, case["rt_lo"], case["rt_hi"])
    return hist, rt, tgt


def _timestamps(case, hist, rt, tgt):
    """One timestamp per K/V row: history and real-time tokens sorted by time, real-time ones the latest and overlapping
    with the exposure times of the candidates."""
    rng = np.random.RandomState(case["lengths_seed"])
    parts = []
    for L, R, T in zip(hist, rt, tgt):
        parts += [np.sort(rng.randint(0, 1000, L)), np.sort(rng.randint(900, 1100, R)), rng.randint(880, 1120, T)]
    return np.concatenate(parts).astype(np.int32)


# --------------------------------------------------------------------------------------------------- state and a pass
def _normal(gen, shape, std=1.0):
    x = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    return x.normal_(0.0, std, generator=gen)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["op"].startswith("gln"):
        return _prepare_gln(case, gen)
    hist, rt, tgt = _lengths(case)
    has_rt = case["rt_hi"] > 0
    full = case["layer"] == "full"
    kv_off = inputs.offsets_from_lengths(hist + rt + tgt)
    q_off = kv_off if full else inputs.offsets_from_lengths(tgt)
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["head_dim"]
    q = _normal(gen, (int(q_off[-1]), Hq, d), case["std"])
    k = _normal(gen, (int(kv_off[-1]), Hkv, d), case["std"])
    v = _normal(gen, (int(kv_off[-1]), Hkv, d), case["std"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    more = {}
    if has_rt:
        more = dict(rt_len=dev(rt), timestamps=dev(_timestamps(case, hist, rt, tgt)), max_rt=int(rt.max()))
    layer = hta.LAYER_FULL if full else hta.LAYER_TARGET
    ints = (dev(q_off), dev(kv_off), dev(hist), dev(tgt), int(hist.max()), int(tgt.max()))
    scale = 1.0 / math.sqrt(d)
    if case["reading"] == "pointwise":
        batch = hta_pw.PointwiseBatch(q, k, v, *ints, scale, 1.0 / float((hist + rt + tgt).max()), layer, **more)
    else:
        batch = hta.Batch(q, k, v, *ints, scale, layer, **more)
    state = dict(op=case["op"], batch=batch)
    if case["op"] == "train":
        batch.prepare_backward()
        state["dout"] = _normal(gen, q.shape)
    return state


def _prepare_gln(case, gen):
    n, d, groups = case["tokens"], case["d_model"], case["groups"]
    cuda = dict(device="cuda", generator=gen)
    gid = torch.randint(0, groups, (n,), dtype=torch.int32, **cuda)
    # groups whose features follow distributions of their own: what group-wise parameters are for
    mean = torch.rand(groups, **cuda) * 2.0 - 1.0
    spread = torch.rand(groups, **cuda) * 1.5 + 0.5
    x = (torch.randn((n, d), **cuda) * spread[gid.long()][:, None] + mean[gid.long()][:, None]).to(torch.bfloat16)
    state = dict(op=case["op"], x=x, gid=gid, gamma=1.0 + 0.2 * torch.randn((groups, d), **cuda),
                 beta=0.2 * torch.randn((groups, d), **cuda), gate=_normal(gen, (n, d)) if case["gated"] else None)
    if case["op"] == "gln_train":
        state["dy"] = _normal(gen, (n, d))
        like = torch.empty_like
        state["y"] = like(x)
        state["out"] = (like(x), like(state["gamma"]), like(state["beta"]), like(x) if case["gated"] else None)
        state["workspace"] = torch.empty(gln.mtfm_gln_bwd_workspace_bytes(d, groups), dtype=torch.uint8, device="cuda")
    return state


EPS = 1e-5


def run(state):
    op = state["op"]
    if op == "gln_infer":
        y, _, _ = gln.mtfm_gln_fwd(state["x"], state["gid"], state["gamma"], state["beta"], EPS, gate=state["gate"],
                                   save_stats=False)
        return {"y": y}
    if op == "gln_train":
        y, mean, rstd = gln.mtfm_gln_fwd(state["x"], state["gid"], state["gamma"], state["beta"], EPS, gate=state["gate"],
                                         y=state["y"])
        dx, dgamma, dbeta, dgate = gln.mtfm_gln_bwd(state["dy"], state["x"], state["gid"], state["gamma"], state["beta"],
                                                    mean, rstd, gate=state["gate"], workspace=state["workspace"],
                                                    out=state["out"])
        return {"y": y, "mean": mean, "rstd": rstd, "dx": dx, "dgamma": dgamma, "dbeta": dbeta, "dgate": dgate}
    batch = state["batch"]
    result = batch.forward()  # (out, lse), or out alone with pointwise weights
    if op == "infer":
        return result
    return result, batch.backward(state["dout"])


# ----------------------------------------------------------------------------------------------- least work of a pass
def work(case):
    if case["op"].startswith("gln"):
        n, d, train, gated = case["tokens"], case["d_model"], case["op"] == "gln_train", case["gated"]
        params = 2 * case["groups"] * d * 4
        size = n * (4 * d + 2 * d * gated + 4) + params             # x (and gate), ids and parameters in, y out
        if train:  # statistics; dy, x (and gate) in, dx (and dgate) out, parameters in, their gradients out
            size += n * (8 + 6 * d + 4 * d * gated + 12) + 2 * params
        return {"bytes": size, "flops": n * d * (25 if train else 8)}
    hist, rt, tgt = (a.astype(np.int64) for a in _lengths(case))
    full = case["layer"] == "full"
    rows = hist + rt + tgt if full else tgt
    # history keys are visible to every row; about half of the real-time keys to the real-time and candidate rows; every
    # row behind the history to itself
    late = rt + tgt if full else tgt
    pairs = int((rows * hist + late * rt // 2 + late).sum()) * case["Hq"]
    d, n_q, n_kv = case["head_dim"], int(rows.sum()) * case["Hq"], int((hist + rt + tgt).sum()) * case["Hkv"]
    lse = 4 * n_q if case["reading"] == "softmax" else 0
    size = 2 * d * (2 * n_q + 2 * n_kv) + lse                       # q, k, v in, out (and lse) out
    flops = 4 * d * pairs                                           # two products per visible pair
    if case["op"] == "train":
        # q, k, v, dout (and out, lse) in; dq, dk, dv out.  Five products: the scores again, dP, dV, dQ, dK.
        size += 2 * d * ((4 if lse else 3) * n_q + 4 * n_kv) + lse
        flops += 10 * d * pairs
    return {"bytes": size, "flops": flops}


def tolerance(case):
    # bf16 results.  Attention also rounds its weights to bf16 between the two products; an element that is a sum of many
    # such terms can be off by a good part of the tensor's root mean square.
    if case["op"].startswith("gln"):
        return {"rel": 4e-3, "max": 2e-2}
    return {"rel": 1e-2, "max": 0.2}
