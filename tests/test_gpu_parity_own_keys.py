"""dK/dV of the targets' own keys: head groups of every remainder of four, in the brief kernels and behind the dQ pass, targets that fill a
workgroup and one more.  Same oracle and bounds as the other parity tests."""
import numpy as np
import pytest

from paper_2602_11235_amd import hta, inputs
from tests.hta_testlib import BRIEF, TWO_PASSES, check_case, close_on_row_scale, form_of
from tests.test_gpu_parity_pointwise import check as check_pointwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,users", [(BRIEF, 4), (TWO_PASSES, 150)])
@pytest.mark.parametrize("heads", [(3, 1, 64), (4, 1, 64), (5, 1, 64), (14, 2, 64), (8, 1, 128), (9, 1, 128), (12, 2, 128), (6, 3, 32), (5, 1, 32)])
def test_heads_of_a_group(form, users, heads):
    hist = np.resize([40, 33, 64, 96], users)
    cfg = inputs.custom_config("own_keys", inputs.LAYER_FULL, hist, np.resize([0, 1, 33, 17], users), *heads, seed=94)
    assert form_of(cfg, hta.CALL_BWD).kind == form
    case = inputs.make_case(cfg)
    check_case(case, with_bwd=True, users=[1, 2, 3], kv_group=0, compare=close_on_row_scale)
    check_pointwise(case, norm=1.0 / 64, users=[1, 2, 3], compare=close_on_row_scale)
