"""Group layer normalization where a token takes a quarter, half or all of a wave's lanes, at the edges of each; groups that end inside one
wave's share, run through several and through all of them; more tokens than the waves take in one pass.  Tolerances are those of
test_gpu_gln.py; a sum over n / groups tokens of float32 terms of order one stays far inside 1e-4 sqrt(n / groups)."""
import numpy as np
import pytest

from oracle import gln_oracle as G
from paper_2602_11235_amd import inputs
from hta_testlib import say
from test_gpu_gln import TOL, TOL_F32, close, run_gpu

pytestmark = pytest.mark.gpu

CASES = [(n, d, groups, dtype, gated)
         for d, groups in ((8, 2), (128, 3), (136, 16), (256, 5), (264, 1), (1016, 4))
         for n, dtype, gated in ((1, "bf16", True), (67, "bf16", False), (1501, "bf16", True), (130, "fp32", True))]
CASES += [(9001, 136, 1, "bf16", True),    # one group: every wave of a workgroup ends in it
          (270001, 8, 3, "bf16", True),    # two passes over the tokens, four tokens side by side
          (135001, 520, 2, "bf16", False)]


@pytest.mark.parametrize("n,d,groups,dtype,gated", CASES)
def test_widths_and_groups(n, d, groups, dtype, gated):
    say(f"  gln n={n} d={d} groups={groups} {dtype} gated={gated}")
    c = inputs.make_gln_case("widths", n, d, groups, dtype=dtype, gated=gated, seed=n % 89 + d)
    if n % 2 and groups > 1:
        c.group_id[: 2 * n // 3] = groups - 1  # two thirds of the tokens in one group, the others everywhere
    got, again = run_gpu(c), run_gpu(c)
    for k, v in got.items():
        assert v is None or np.array_equal(v, again[k]), f"{k} differs between two runs"
    y, mean, rstd = G.forward(c.x, c.group_id, c.gamma, c.beta, c.eps, c.gate)
    dx, dgamma, dbeta, du = G.backward(c.dy, c.x, c.group_id, c.gamma, c.beta, c.eps, c.gate)
    tol = 1e-4 * max(1., np.sqrt(n / groups))
    for k, ref, t in (("y", y, TOL[dtype]), ("mean", mean, TOL_F32), ("rstd", rstd, TOL_F32), ("dx", dx, TOL[dtype]),
                      ("dgamma", dgamma, (tol, 1e-4)), ("dbeta", dbeta, (tol, 1e-4)), ("du", du, TOL[dtype])):
        if ref is not None:
            close(k, got[k], ref, t)
