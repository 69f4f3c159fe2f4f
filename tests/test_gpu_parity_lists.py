"""dK/dV from work lists of which a few long users hold much of the work: their key tiles are dealt to several lists, and items of one iteration, of a
few and of hundreds follow each other.  Same oracle and bounds as the other parity tests."""
import numpy as np
import pytest

from paper_2602_11235_amd import hta, inputs
from tests.hta_testlib import ONE_PASS, TWO_PASSES, check_case, close_on_row_scale, form_of
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


# Kernels that keep a user: histories, heads, form.  In one pass the next item is taken with the start of an item, where no history has six blocks of
# 32 keys, or six blocks before its end; with the rows resident, with the first wave's last 384 keys.  Users without history or targets among them.
KEPT = {
    "one_pass_early": ([160, 0, 129, 1, 160, 33], (8, 2, 64), ONE_PASS),
    "one_pass_late": ([161, 0, 160, 192, 1, 193, 224, 225, 400], (8, 2, 64), ONE_PASS),
    "resident": ([1153, 0, 1537, 383, 1152, 1, 1536, 769], (6, 2, 64), TWO_PASSES),
}


@pytest.mark.parametrize("name", KEPT)
def test_the_next_item_of_a_kernel_that_keeps_a_user(name):
    hist, heads, kind = KEPT[name]
    n = 701
    cfg = inputs.custom_config(name, inputs.LAYER_TARGET, np.resize(hist, n), np.resize([40, 3, 0, 17, 33], n), *heads, seed=94)
    form = form_of(cfg, hta.CALL_BWD)
    assert form.kind == kind and (kind == ONE_PASS or (form.ways, form.option) == (0, 1))
    users = sorted(set(range(20)) | set(range(0, n, 40)) | {n - 1})
    check_case(inputs.make_case(cfg), with_bwd=True, users=users, compare=close_on_row_scale)
