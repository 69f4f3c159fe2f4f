"""The library's calls can be captured into a HIP graph (they only enqueue kernels: no allocation, no memset, no
synchronisation) and a replay returns what the eager call returns, every time: replays are interleaved with eager
work and synchronisations, and each one is compared bit for bit with the eager result."""
import numpy as np
import pytest
import torch

from paper_2602_11235_amd import gln, inputs
from tests.hta_testlib import backward_kernels, device_batch, say, to_torch

pytestmark = pytest.mark.gpu


def _replay_and_compare(graph, outputs, eager, disturb):
    for i in range(4):
        for t in outputs:
            t.fill_(float("nan")) if t.is_floating_point() else t.zero_()
        disturb()                       # eager work of the same library between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, t, ref in zip(("out", "lse", "dq", "dk", "dv"), outputs, eager):
            assert torch.equal(t, ref), f"replay {i}: {name} differs from the eager result"


# a few users: forward and backward in their forms for calls of little work
FEW = inputs.custom_config("few", inputs.LAYER_TARGET, [300, 65, 1000], [7, 33, 40], 8, 2, 64, seed=43, rt_len=[40, 0, 70])

# many users of few query rows: the backward in one kernel, more items than workgroups; and a full layer with real-time tokens
ONE_PASS = {
    "one_pass": inputs.custom_config("one_pass", inputs.LAYER_TARGET, np.resize([300, 129, 0, 257], 600), np.resize([64, 33, 48], 600), 8, 2,
                                     64, seed=44),
    "one_pass_full_rt": inputs.custom_config("one_pass_full_rt", inputs.LAYER_FULL, np.resize([330, 289, 256, 0, 200], 600),
                                             np.resize([60, 33, 0], 600), 4, 4, 64, seed=45, rt_len=np.resize([0, 5, 33, 40], 600)),
}


@pytest.mark.parametrize("name, with_bwd", [*((name, True) for name in ONE_PASS), ("I1", False), ("I2_RT", False), ("I3", False), ("C2", True), ("C2_RT", True), ("few", True)])
def test_forward_and_backward_replay_from_a_graph(name, with_bwd):
    say(f"[graph] {name} bwd={with_bwd}")
    case = inputs.make_case(FEW if name == "few" else ONE_PASS.get(name) or inputs.CONFIGS[name])
    b = device_batch(case)
    other = device_batch(inputs.make_case(inputs.custom_config("other", inputs.LAYER_FULL, [300, 65], [7, 33], 8, 2, 64, seed=41)))
    dout = to_torch(case.dout, case.cfg.dtype)
    b.forward()
    if with_bwd:                        # warm-up: every one-time query of the library happens outside the capture
        kernels = backward_kernels(lambda: b.backward(dout))
        assert (kernels == (1, 0)) == (name in ONE_PASS), kernels
    torch.cuda.synchronize()
    outputs = [b.out, b.lse] + ([b.dq, b.dk, b.dv] if with_bwd else [])
    eager = [t.clone() for t in outputs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.forward()
        if with_bwd:
            b.backward(dout)
    _replay_and_compare(graph, outputs, eager, lambda: other.forward())


# Requests whose lengths are rewritten between the replays of one graph, captured with bounds that hold for all of them: the longest user as long as
# the bound, then a third of it, then one without keys.  (Same totals, which are the graph's.)
LENGTHS = ([8192, 64, 36], [2764, 2764, 2764], [4100, 0, 4192]), ([64, 1, 31], [32, 32, 32], [5, 60, 31])


@pytest.mark.parametrize("heads", [(8, 2, 64), (16, 2, 128)])
def test_replays_go_by_the_lengths(heads):
    say(f"[graph] lengths {heads}")
    cases = [inputs.make_case(inputs.custom_config("lengths", inputs.LAYER_TARGET, hist, targets, *heads, seed=46)) for hist, targets in zip(*LENGTHS)]
    batches = [device_batch(c) for c in cases]
    for b in batches:
        b.max_hist, b.max_targets = 8192, 64     # (the workspace of the first, which has these, serves all)
        b.fwd_workspace, b.fwd_workspace_bytes = batches[0].fwd_workspace, batches[0].fwd_workspace_bytes
    eager = [tuple(t.clone() for t in b.forward()) for b in batches]
    captured = batches[0]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured.forward()
    for i in (1, 2, 0, 1):
        source = device_batch(cases[i])
        for name in ("q", "k", "v", "q_offsets", "kv_offsets", "hist_len", "n_targets"):
            getattr(captured, name).copy_(getattr(source, name))
        captured.out.zero_(), captured.lse.zero_()
        batches[2].forward()                     # eager work between the replays, in the same workspace
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t, ref in zip((captured.out, captured.lse), eager[i]):
            assert torch.equal(t, ref), f"lengths {i}"


def test_group_layer_normalization_replays_from_a_graph():
    say("[graph] gln")
    c = inputs.make_gln_case("g", 3000, 512, 8, dtype="bf16", gated=True, seed=42)
    dev = lambda a, bf=False: (lambda t: t.to(torch.bfloat16) if bf else t)(torch.from_numpy(np.ascontiguousarray(a)).to("cuda"))
    x, u, dy = dev(c.x, True), dev(c.gate, True), dev(c.dy, True)
    gid, gamma, beta = dev(c.group_id), dev(c.gamma), dev(c.beta)
    y = torch.empty_like(x)
    mean = torch.empty(x.shape[0], device="cuda")
    out = (torch.empty_like(x), torch.empty_like(gamma), torch.empty_like(gamma), torch.empty_like(x))
    ws = torch.empty(gln.mtfm_gln_bwd_workspace_bytes(512, 8), dtype=torch.uint8, device="cuda")

    stats = {}

    def run():
        _, stats["mean"], stats["rstd"] = gln.mtfm_gln_fwd(x, gid, gamma, beta, c.eps, gate=u, y=y)
        gln.mtfm_gln_bwd(dy, x, gid, gamma, beta, stats["mean"], stats["rstd"], gate=u, workspace=ws, out=out)

    run()
    torch.cuda.synchronize()
    eager_y, eager_dx, eager_du = y.clone(), out[0].clone(), out[3].clone()
    eager_dgamma = out[1].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for i in range(4):
        y.zero_(); out[0].zero_(); out[1].zero_(); out[3].zero_()
        gln.mtfm_gln_fwd(x[:100], gid[:100], gamma, beta, c.eps)   # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, eager_y) and torch.equal(out[0], eager_dx) and torch.equal(out[3], eager_du), f"replay {i}"
        # the workgroup sums use LDS atomics: equal up to the order of float32 additions
        assert torch.allclose(out[1], eager_dgamma, rtol=1e-5, atol=1e-5), f"replay {i}: dgamma"
