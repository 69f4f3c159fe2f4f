"""How the backward kernels with a work queue deal out their work: host rules on sizes, asked without a GPU."""
import ctypes

import pytest

from paper_2602_11235_amd import hta
from tests import test_gpu_parity_lists as lists
from tests.hta_testlib import ONE_PASS, TWO_PASSES, form_of_sizes

HEADS = (8, 2, 64)


def lists_of_sizes(batch, total_q, total_kv, max_hist, max_targets, heads, layer, max_rt=0):
    block = hta._HTA_BLOCK.pack(*[0] * 13, int(max_rt > 0), 0, 0, 0, total_q, total_kv, batch, max_hist, max_rt, max_targets, *heads, 1.0, 1.0,
                                hta.BF16, layer, hta.CALL_BWD)
    out = (ctypes.c_int32 * 2)()
    assert hta.load_library().mtfm_binding_hta_lists(block, out) == hta.OK
    return tuple(out)


@pytest.mark.parametrize("users,longest,mean,late", [(463, 156, 98, 0), (1565, 96, 72, 0), (227, 1275, 796, 1), (562, 444, 250, 1)])
def test_late_requests_do_not_follow_the_bounds(users, longest, mean, late):
    """Users of few blocks of keys ask for the next item with their start, whatever the bounds of the call."""
    for loose in (1, 4, 16):
        sizes = (users, users * 20, users * (mean + 20), longest * loose, 32, HEADS, hta.LAYER_TARGET)
        assert loose > 1 or form_of_sizes(hta.CALL_BWD, *sizes).kind == ONE_PASS
        assert lists_of_sizes(*sizes)[0] == late


@pytest.mark.parametrize("name", lists.SHAPES)
def test_shapes_whose_tiles_go_to_four_lists(name):
    cfg = lists.config(name)
    hist, targets, rt = cfg.hist[1], cfg.targets[1], [0] * cfg.batch if cfg.rt is None else cfg.rt[1]
    total = sum(hist) + sum(targets) + sum(rt)
    sizes = (cfg.batch, total, total, max(hist), max(targets), (cfg.Hq, cfg.Hkv, cfg.head_dim), cfg.layer, max(rt))
    assert form_of_sizes(hta.CALL_BWD, *sizes)[:3] == (TWO_PASSES, 0, 0) and lists_of_sizes(*sizes)[1] == 2


@pytest.mark.parametrize("users,longest,mean", [(256, 1024, 768), (60, 1000, 900), (200, 8192, 1500), (40, 900, 400)])
def test_users_alike_many_or_short_stay_on_one_list(users, longest, mean):
    total = users * (mean + 32)
    assert lists_of_sizes(users, total, total, longest, 64, HEADS, hta.LAYER_FULL)[1] == 0
