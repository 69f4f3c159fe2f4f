"""Shares of dgamma, dbeta: as many workgroups as the tokens allow, and their sum at the edges of its split (a lane has every 64th share, at most four).
A workgroup takes 8 tokens where tokens lie side by side and are few, 16 at 512 features, 8 with more; the workspace shows how many wrote a share.
float32 sums of n / groups terms of order one, each within 2^-24 of its size: far inside 1e-4 sqrt(n / groups)."""
import numpy as np
import pytest
import torch

from oracle import gln_oracle as G
from paper_2602_11235_amd import gln, inputs
from hta_testlib import say
from test_gpu_gln import close, dev, host

pytestmark = pytest.mark.gpu

MOST = 256


@pytest.mark.parametrize("shares", [1, 2, 63, 64, 65, 128, 129, 192, 193, 255, 256, 400])
@pytest.mark.parametrize("d,groups,dtype,tokens", [(8, 1, "fp32", 8), (24, 3, "bf16", 8), (128, 2, "bf16", 8), (136, 4, "fp32", 8), (256, 2, "bf16", 8),
                                                   (264, 2, "bf16", 16), (520, 2, "fp32", 8)])
def test_shares_and_their_sum(shares, d, groups, dtype, tokens):
    n = tokens * shares - 3
    say(f"  gln shares={shares} d={d} groups={groups} {dtype} n={n}")
    c = inputs.make_gln_case("shares", n, d, groups, dtype=dtype, gated=True, seed=shares)
    x, dy, u, gid, gamma, beta = dev(c.x, dtype), dev(c.dy, dtype), dev(c.gate, dtype), dev(c.group_id), dev(c.gamma), dev(c.beta)
    _, mean, rstd = gln.mtfm_gln_fwd(x, gid, gamma, beta, c.eps, gate=u)
    workspace = torch.full((gln.mtfm_gln_bwd_workspace_bytes(d, groups) // 4,), float("nan"), device="cuda")
    _, dgamma, dbeta, _ = gln.mtfm_gln_bwd(dy, x, gid, gamma, beta, mean, rstd, gate=u, workspace=workspace.view(torch.uint8))
    written = torch.isfinite(workspace).view(-1, 2 * groups * d)
    assert bool((written.all(1) == written.any(1)).all())
    assert int(written.any(1).sum()) == min(shares, MOST)
    _, want_gamma, want_beta, _ = G.backward(c.dy, c.x, c.group_id, c.gamma, c.beta, c.eps, c.gate)
    tol = 1e-4 * max(1., np.sqrt(n / groups))
    close("dgamma", host(dgamma), want_gamma, (tol, 1e-4))
    close("dbeta", host(dbeta), want_beta, (tol, 1e-4))


@pytest.mark.parametrize("d,last", [(128, 16384), (256, 8192)])
def test_the_last_call_of_few_tokens_and_the_next(d, last):
    """Eight waves to a workgroup up to `last` tokens, sixteen beyond."""
    for n in (last, last + 1):
        say(f"  gln n={n} d={d}")
        c = inputs.make_gln_case("few", n, d, 5, dtype="bf16", gated=True, seed=n % 97)
        x, dy, u, gid, gamma, beta = dev(c.x, "bf16"), dev(c.dy, "bf16"), dev(c.gate, "bf16"), dev(c.group_id), dev(c.gamma), dev(c.beta)
        _, mean, rstd = gln.mtfm_gln_fwd(x, gid, gamma, beta, c.eps, gate=u)
        dx, dgamma, dbeta, du = gln.mtfm_gln_bwd(dy, x, gid, gamma, beta, mean, rstd, gate=u)
        want = G.backward(c.dy, c.x, c.group_id, c.gamma, c.beta, c.eps, c.gate)
        tol = 1e-4 * np.sqrt(n / 5)
        for name, got, ref, t in (("dx", dx, want[0], (2e-2, 2e-2)), ("dgamma", dgamma, want[1], (tol, 1e-4)), ("dbeta", dbeta, want[2], (tol, 1e-4)),
                                  ("du", du, want[3], (2e-2, 2e-2))):
            close(name, host(got), ref, t)
