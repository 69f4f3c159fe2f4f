"""Which kernels a call takes: host rules on sizes, asked without a GPU.  (That the kernels are right is what the parity tests check.)"""
import pytest

from paper_2602_11235_amd import hta
from tests.hta_testlib import BRIEF, TWO_PASSES, form_of_sizes

HEADS = (8, 2, 64)


def target_layer(call, users, keys, candidates, heads=HEADS, loose=1, max_rt=0):
    """users of one length; bounds of the keys `loose` times that"""
    return form_of_sizes(call, users, users * candidates, users * (keys + max_rt + candidates), keys * loose, candidates, heads, hta.LAYER_TARGET,
                         max_rt * loose)


@pytest.mark.parametrize("call", [hta.CALL_FWD, hta.CALL_PW_FWD])
def test_forward_forms(call):
    assert target_layer(call, 1, 2048, 128).kind > 1                 # one request: its keys in several pieces
    assert target_layer(call, 40, 500, 16).kind == 1                 # a unit for every 32 rows: in one
    assert target_layer(call, 2000, 500, 16).kind == 0               # a full chip: the ordinary kernel ...
    assert target_layer(call, 2000, 500, 16).schedule == 0           # ... on users of one length, as they are given
    assert target_layer(call, 2000, 500, 16, max_rt=50).schedule == 1


@pytest.mark.parametrize("call", [hta.CALL_BWD, hta.CALL_PW_BWD])
def test_backward_forms(call):
    assert target_layer(call, 4, 300, 60).kind == BRIEF
    assert target_layer(call, 277, 241, 3).kind == BRIEF
    assert target_layer(call, 1000, 1500, 70, heads=(12, 2, 64)).kind == TWO_PASSES


@pytest.mark.parametrize("users", [65, 129, 300])
def test_many_users_do_not_stand_in_a_list(users):
    """Every wave of a list looks at all lengths, 64 at a time, which many users do not repay."""
    form = target_layer(hta.CALL_FWD, users, 100, 2, heads=(4, 1, 64))
    assert form.kind == 1 and form.option == 1


@pytest.mark.parametrize("users,keys,candidates,heads", [(4, 149, 2, (16, 2, 128)), (3, 340, 11, (8, 1, 64)), (2, 719, 53, (16, 4, 64)), (3, 192, 1, (16, 4, 64))])
def test_little_work_is_shared_by_four_waves(users, keys, candidates, heads):
    """With a wave to each key block these take 1.15 to 1.3 times as long: the chip is nearly empty, and one wave's chain is the time."""
    assert target_layer(hta.CALL_BWD, users, keys, candidates, heads)[:2] == (BRIEF, 4)


@pytest.mark.parametrize("users,keys,candidates,heads", [(11, 384, 114, (8, 1, 64)), (8, 126, 84, (4, 1, 64)), (13, 99, 84, (8, 1, 128)), (60, 400, 10, HEADS)])
def test_brief_form_does_not_follow_the_bounds(users, keys, candidates, heads):
    """Bounds far above the lengths made the chains of dQ seem to be the time, and up to twice of it was lost."""
    assert len({target_layer(hta.CALL_BWD, users, keys, candidates, heads, loose)[:2] for loose in (1, 4, 16)}) == 1
