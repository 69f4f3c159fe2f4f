"""Which kernels a call takes: host rules on sizes, asked without a GPU.  (That the kernels are right is what the parity tests check.)"""
import pytest

from paper_2602_11235_amd import hta
from tests import test_gpu_parity_inference as requests, test_gpu_parity_shapes as shapes
from tests.hta_testlib import BRIEF, ONE_PASS, TWO_PASSES, form_of, form_of_sizes

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


# What the parity tests' shapes are there for: a prefix of the name -> (kind, waves per key block, option) of the backward pass
BACKWARD = {"brief_alone_d32": (BRIEF, 1, 1), "brief_alone_long": (BRIEF, 1, 1), "brief_alone": (BRIEF, 1, 0), "brief": (BRIEF, 4, 0),
            "one_way": (TWO_PASSES, 1, 0), "two_ways": (TWO_PASSES, 2, 0), "four_ways": (TWO_PASSES, 4, 0), "one_pass": (ONE_PASS, 0, 0),
            "rows_resident": (TWO_PASSES, 0, 1), "ordinary": (TWO_PASSES, 0, 0), "two_row_blocks": (TWO_PASSES, 0, 0)}


@pytest.mark.parametrize("name", shapes.SHAPES)
def test_shapes_run_the_kernels_they_name(name):
    cfg = shapes.config(name)
    for weights in ("softmax", "pointwise") if name in shapes.POINTWISE else ("softmax",):
        forward, backward = [form_of(cfg, call) for call in ((hta.CALL_FWD, hta.CALL_BWD) if weights == "softmax" else (hta.CALL_PW_FWD, hta.CALL_PW_BWD))]
        if name.startswith("rows64"):  # requests, two blocks of 32 rows to a workgroup
            assert forward.ways == 2 and (forward.kind > 1 if name.endswith("long") else forward.kind == 1)
        else:
            assert backward[:3] == next(BACKWARD[k] for k in BACKWARD if name.startswith(k))


@pytest.mark.parametrize("name,ways,schedule", [("four_ways", 4, 0), ("four_ways_many", 4, 0), ("two_ways", 2, 0), ("one_way", 1, 0), ("queue_one_pass", 0, 1),
                                                ("queue", 0, 1)])
def test_users_of_one_length_go_without_the_schedule(name, ways, schedule):
    cfg = shapes.config_of_one_length(name)
    assert form_of(cfg, hta.CALL_FWD).schedule == 0
    backward = form_of(cfg, hta.CALL_BWD)
    assert backward.kind == (ONE_PASS if name == "queue_one_pass" else TWO_PASSES) and (backward.ways, backward.schedule) == (ways, schedule)


# (pieces, row blocks, grid); pieces: one, or more than one
LIST_FORMS = {"many_users": (1, 1, 1), "a_lane_more": (1, 1, 1), "three_waves_of_users": (1, 1, 1), "pieces_grow": (2, 1, 0), "more_than_units": (1, 2, 0),
              "two_row_blocks_d128": (1, 2, 0), "two_row_blocks_d128_in_pieces": (2, 2, 0), "two_row_blocks_d128_full": (1, 2, 0), "many_pieces": (2, 1, 0)}


@pytest.mark.parametrize("call", [hta.CALL_FWD, hta.CALL_PW_FWD])
@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("name", requests.LISTS)
def test_lists_run_the_form_they_name(name, with_rt, call):
    form = form_of(requests.config_of_list(name, with_rt), call)
    assert (min(form.kind, 2), form.ways, form.option) == LIST_FORMS[name]


@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("heads", [(8, 2, 64), (3, 1, 64), (16, 2, 128), (4, 2, 32)])
def test_long_histories_are_split_over_workgroups(heads, with_rt):
    assert form_of(requests.config_of_long(heads, with_rt), hta.CALL_FWD).kind > 1
