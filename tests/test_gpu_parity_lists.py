"""dK/dV from work lists of which a few long users hold much of the work: their key tiles are dealt to several lists, and items of one iteration, of a
few and of hundreds follow each other.  Same oracle and bounds as the other parity tests."""
import numpy as np
import pytest

from paper_2602_11235_amd import hta, inputs
from tests.hta_testlib import TWO_PASSES, check_case, close_on_row_scale, form_of
from tests.test_gpu_parity_pointwise import check as check_pointwise

pytestmark = pytest.mark.gpu

SHAPES = {  # users, history of every fourth user, real-time tokens, heads
    "d64": (60, 3000, False, (8, 2, 64)),
    "d64_rt": (60, 3000, True, (8, 2, 64)),
    "d128": (40, 1500, False, (16, 2, 128)),
    "d128_rt": (40, 1500, True, (16, 2, 128)),
    "d32": (44, 4000, True, (4, 2, 32)),
}


def config(name):
    n, longest, rt, heads = SHAPES[name]
    hist = np.where(np.arange(n) % 4 == 3, longest + np.resize([0, 1, 63, 65], n), np.resize([0, 1, 31, 33, 127, 128, 129, 256, 300], n))
    return inputs.custom_config(name, inputs.LAYER_FULL, hist, np.resize([3, 0, 17, 40], n), *heads, seed=93,
                                rt_len=np.resize([0, 1, 33, 64], n) if rt else None)


@pytest.mark.parametrize("name", SHAPES)
def test_long_users_among_short_ones(name):
    cfg = config(name)
    for call in (hta.CALL_BWD, hta.CALL_PW_BWD):
        form = form_of(cfg, call)
        assert (form.kind, form.ways, form.option) == (TWO_PASSES, 0, 0)  # the kernels with a work queue
    case = inputs.make_case(cfg)
    users = [0, 1, 2, 3, 4, 5, 6, 8, 16, 26]
    check_case(case, with_bwd=True, users=users, kv_group=1, compare=close_on_row_scale)
    check_pointwise(case, norm=1.0 / 64, users=users[:3] + users[4:], compare=close_on_row_scale)
