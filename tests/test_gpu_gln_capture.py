"""A call of the group layer normalization can be captured though it is the first of its kernels in the process (run by itself, this file is that)."""
import pytest
import torch

from paper_2602_11235_amd import gln, inputs
from hta_testlib import say
from test_gpu_gln import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,groups,dtype,gated", [(2040, 4, "fp32", True), (1536, 2, "bf16", False), (120, 16, "fp32", True), (248, 3, "bf16", True)])
def test_first_call_in_a_capture(d, groups, dtype, gated):
    say(f"  gln capture d={d} groups={groups} {dtype} gated={gated}")
    n = 301
    c = inputs.make_gln_case("capture", n, d, groups, dtype=dtype, gated=gated, seed=d)
    x, dy, u = dev(c.x, dtype), dev(c.dy, dtype), dev(c.gate, dtype) if gated else None
    gid, gamma, beta = dev(c.group_id), dev(c.gamma), dev(c.beta)
    y, stats = torch.empty_like(x), (torch.empty(n, device="cuda"), torch.empty(n, device="cuda"))
    out = (torch.empty_like(x), torch.empty_like(gamma), torch.empty_like(beta), torch.empty_like(x) if gated else None)
    workspace = torch.empty(gln.mtfm_gln_bwd_workspace_bytes(d, groups), dtype=torch.uint8, device="cuda")

    def step():
        gln.mtfm_gln_fwd(x, gid, gamma, beta, c.eps, gate=u, y=y, stats=stats)
        gln.mtfm_gln_bwd(dy, x, gid, gamma, beta, *stats, gate=u, workspace=workspace, out=out)

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    results = [t for t in (y, *stats, *out) if t is not None]
    step()
    torch.cuda.synchronize()
    eager = [t.clone() for t in results]
    for _ in range(3):
        for t in results:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(t, e) for t, e in zip(results, eager))
        step()
