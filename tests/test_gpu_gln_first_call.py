"""The first call of the group layer normalization in a process may be a backward pass, and calls of other kernels work behind it."""
import os
import subprocess
import sys

import pytest

from paper_2602_11235_amd import gln

pytestmark = pytest.mark.gpu

PROGRAM = """
import torch
from paper_2602_11235_amd import gln
for d, groups in ((64, 3), (512, 16), (2048, 2)):
    n = 100
    x, dy = torch.randn(n, d, device="cuda"), torch.randn(n, d, device="cuda")
    gid = torch.randint(0, groups, (n,), dtype=torch.int32, device="cuda")
    gamma, beta = torch.ones(groups, d, device="cuda"), torch.zeros(groups, d, device="cuda")
    mean, rstd = x.mean(1), (x.var(1, unbiased=False) + 1e-5).rsqrt()
    _, dgamma, dbeta, _ = gln.mtfm_gln_bwd(dy, x, gid, gamma, beta, mean, rstd)
    want = torch.zeros(groups, d, device="cuda").index_add_(0, gid.long(), dy)
    assert torch.allclose(dbeta, want, atol=1e-4), d
    y, _, _ = gln.mtfm_gln_fwd(x, gid, gamma, beta, 1e-5)
    assert torch.allclose(y, (x - mean[:, None]) * rstd[:, None], atol=1e-4), d
print("done")
"""


def test_backward_first():
    root = os.path.dirname(os.path.dirname(os.path.abspath(gln.__file__)))
    result = subprocess.run([sys.executable, "-c", PROGRAM], cwd=root, capture_output=True, text=True, timeout=100)
    assert result.returncode == 0 and result.stdout.endswith("done\n"), result.stderr[-2000:]
