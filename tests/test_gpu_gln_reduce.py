"""The sum of the workgroups' shares of dgamma, dbeta at the edges of its split: shares per lane, columns per workgroup.
float32 sums of n / groups terms of order one per element, each within 2^-24 of its size: far inside 1e-4 sqrt(n / groups)."""
import numpy as np
import pytest

from oracle import gln_oracle as G
from paper_2602_11235_amd import inputs
from hta_testlib import say
from test_gpu_gln import close, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shares", [1, 2, 63, 64, 65, 128, 449, 511, 512])   # 8 tokens each; a lane has every 64th
@pytest.mark.parametrize("d,groups", [(8, 1), (8, 2), (16, 1), (24, 3), (520, 2)])   # 2 d groups columns, 32 per workgroup
def test_sum_of_the_shares(shares, d, groups):
    n = 8 * shares - 3 if shares > 1 else 5
    say(f"  gln shares={shares} d={d} groups={groups} n={n}")
    c = inputs.make_gln_case("reduce", n, d, groups, dtype="fp32", gated=True, seed=shares)
    got = run_gpu(c)
    _, dgamma, dbeta, _ = G.backward(c.dy, c.x, c.group_id, c.gamma, c.beta, c.eps, c.gate)
    tol = 1e-4 * max(1., np.sqrt(n / groups))
    close("dgamma", got["dgamma"], dgamma, (tol, 1e-4))
    close("dbeta", got["dbeta"], dbeta, (tol, 1e-4))
