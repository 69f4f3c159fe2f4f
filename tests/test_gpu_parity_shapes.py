"""GPU parity at the shapes between which the library chooses: users, rows and histories small, middling and many, so that
every form of the forward, dQ and dK/dV passes runs on lengths at the edges of its tiles.  Same oracle and bounds as the
other parity tests."""
import numpy as np
import pytest
import torch

from paper_2602_11235_amd import inputs
from tests.hta_testlib import check_case, close_on_row_scale, device_batch, queue_takes, say, to_torch
from tests.test_gpu_parity_pointwise import check as check_pointwise

pytestmark = pytest.mark.gpu
FULL, TARGET = inputs.LAYER_FULL, inputs.LAYER_TARGET

HIST = np.array([0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 200])
TGTS = np.array([0, 1, 7, 8, 9, 16, 31, 32, 33, 40])
RT = np.array([0, 1, 31, 32, 33, 65])
cycle = lambda values, n: np.resize(values, n)

# name: layer, users, history beyond HIST (in a tuple: of every fourth user), targets beyond TGTS, heads, with real-time tokens
SHAPES = {
    # a few dozen users: the rows of 32 keys, and the keys of 32 rows, shared by the waves of a workgroup
    "brief": (FULL, 12, 0, 0, (8, 2, 64), False),
    "brief_rt": (TARGET, 24, 0, 0, (8, 2, 64), True),
    "brief_d32": (FULL, 16, 0, 0, (3, 1, 32), True),
    "brief_d128": (TARGET, 20, 0, 0, (6, 2, 128), True),
    # ... and few rows against more keys: a wave to each key block, dQ behind dK/dV or (d32, long) in front
    "brief_alone": (TARGET, 100, 200, 0, (8, 2, 64), False),
    "brief_alone_d32": (TARGET, 90, 100, 0, (6, 2, 32), False),
    "brief_alone_d128": (TARGET, 40, 600, 0, (16, 2, 128), True),
    "brief_alone_long": (TARGET, 70, 800, 0, (8, 2, 64), True),
    # more of them: dQ in its ordinary form, a key block's rows shared by one, two or four waves
    "one_way": (TARGET, 330, 0, 0, (8, 2, 64), False),
    "one_way_rt": (TARGET, 330, 0, 0, (6, 2, 64), True),
    "one_way_many_rt": (TARGET, 1500, 100, 0, (6, 2, 64), True),
    "one_way_single_heads_long": (FULL, 400, (500,), 0, (4, 4, 64), False),
    "one_pass_single_heads": (FULL, 400, 0, 0, (4, 4, 64), False),
    "two_ways": (FULL, 160, 0, 0, (8, 2, 64), False),
    "two_ways_rt": (FULL, 160, 0, 0, (8, 2, 64), True),
    "four_ways": (FULL, 64, 0, 0, (8, 2, 64), True),
    "four_ways_d128": (FULL, 40, 0, 0, (16, 2, 128), True),
    # 64 rows per workgroup in the forward pass of some requests, keys in one piece and (long) in several
    "rows64": (TARGET, 20, 500, 70, (8, 2, 64), True),
    "rows64_d128": (TARGET, 16, 700, 30, (16, 2, 128), False),
    "rows64_d128_rt": (TARGET, 16, 700, 30, (16, 2, 128), True),
    "rows64_long": (TARGET, 10, (8000,), 100, (8, 2, 64), True),
    "rows64_d128_long": (TARGET, 10, (6000,), 60, (16, 2, 128), True),
    # enough for the ordinary dK/dV pass; blocks behind the history in its grid (in a launch of their own at 128)
    "ordinary_d32": (FULL, 400, 500, 0, (4, 2, 32), False),
    "ordinary_d32_rt": (FULL, 400, 500, 0, (4, 2, 32), True),
    "ordinary_d128_rt": (FULL, 160, 500, 0, (16, 2, 128), True),
    "two_row_blocks": (FULL, 40, 2048, 0, (8, 2, 64), False),
    # few query rows per user against long histories: the whole backward in one kernel, or (r not a power of two) dK/dV with a
    # user's rows resident in LDS
    "one_pass": (TARGET, 256, 512, 88, (8, 2, 64), False),
    "rows_resident": (TARGET, 256, 512, 88, (6, 2, 64), False),
    "rows_resident_r6": (TARGET, 300, 800, 20, (12, 2, 64), False),
    # groups of more query heads than a tile has lanes, cut into chunks of which the last one is not full; all forms again
    "brief_wide": (TARGET, 6, 0, 0, (40, 1, 64), True),
    "brief_wide_d32": (TARGET, 5, 0, 0, (130, 1, 32), False),
    "brief_wide_d128": (TARGET, 4, 0, 0, (66, 2, 128), False),
    "rows64_wide": (TARGET, 2, 1000, 100, (70, 1, 64), True),
    "rows64_wide_d128": (TARGET, 2, 2500, 100, (70, 1, 128), False),
    "rows64_wider": (TARGET, 2, 300, 40, (130, 1, 64), False),
    "rows64_wider_d128": (TARGET, 2, 300, 40, (130, 1, 128), True),
    "four_ways_wide_d32": (FULL, 24, 0, 0, (130, 1, 32), True),
    "four_ways_wide": (FULL, 10, 0, 0, (300, 1, 64), True),
    "four_ways_wide_d128": (FULL, 24, 0, 0, (130, 1, 128), False),
    "ordinary_wide_d128_rt": (FULL, 40, 500, 0, (33, 1, 128), True),
}


def config(name):
    layer, n, more_hist, more_tgts, (Hq, Hkv, d), rt = SHAPES[name]
    if isinstance(more_hist, tuple):
        more_hist = np.where(np.arange(n) % 4 == 3, more_hist[0], 0)
    return inputs.custom_config(name, layer, cycle(HIST, n) + more_hist, cycle(TGTS, n) + more_tgts, Hq, Hkv, d, dtype="bf16",
                                std=0.3, seed=77, rt_len=cycle(RT, n) if rt else None)


def make(name):
    n = SHAPES[name][1]
    return inputs.make_case(config(name)), sorted(set(range(0, n, max(1, n // 24))) | {1, n - 1}) if n > 64 else None


@pytest.mark.parametrize("name", SHAPES)
def test_shapes(name):
    case, users = make(name)
    check_case(case, with_bwd=True, users=users, compare=close_on_row_scale)


# users of one length, which the library takes in the order given (no launch that orders them): a few long tiles, a key block's rows shared by
# four, two and one waves; and kernels with a work queue (one pass, head_dim 32), which have theirs cleared by that launch
ONE_LENGTH = {
    "four_ways": (FULL, 60, 200, 20, (8, 2, 64)),
    "four_ways_many": (FULL, 160, 129, 33, (8, 2, 64)),
    "two_ways": (FULL, 160, 129, 20, (8, 2, 64)),
    "one_way": (TARGET, 300, 500, 20, (16, 2, 128)),
    "queue_one_pass": (FULL, 400, 65, 7, (6, 6, 64)),
    "queue": (FULL, 500, 520, 9, (4, 2, 32)),
}


def config_of_one_length(name):
    layer, users, hist, targets, heads = ONE_LENGTH[name]
    return inputs.custom_config("one_length", layer, np.full(users, hist), np.full(users, targets), *heads, seed=78)


@pytest.mark.parametrize("name", ONE_LENGTH)
def test_users_of_one_length(name):
    case = inputs.make_case(config_of_one_length(name))
    check_case(case, with_bwd=True, users=[0, 1, case.batch // 2, case.batch - 1], compare=close_on_row_scale)


@pytest.mark.parametrize("name", ["rows_resident", "rows_resident_r6"])
def test_the_resident_shapes_reach_the_resident_kernel(name):
    """By the takes from the work queue: one item per (user, kv head) there, one per 128 keys of the longest in the kernel that streams the
    rows, and the kernels that share a block's rows between waves have no queue."""
    case, _ = make(name)
    batch = device_batch(case)
    batch.forward()
    batch.backward(to_torch(case.dout, "bf16"))
    items, units = case.batch * case.cfg.Hkv, torch.cuda.get_device_properties(0).multi_processor_count
    taken = queue_takes(batch)
    say(f"    {items} items, {taken} takes")
    assert units < items and 0 < taken < items + 2 * units


POINTWISE = ["brief_rt", "brief_d128", "brief_alone_long", "one_way_rt", "two_ways_rt", "four_ways", "rows64", "rows64_d128_rt", "rows64_d128_long",
             "ordinary_d32_rt", "brief_wide", "rows64_wide", "rows64_wider_d128"]


@pytest.mark.parametrize("name", POINTWISE)
def test_shapes_with_pointwise_weights(name):
    case, users = make(name)
    check_pointwise(case, norm=1.0 / 64, users=users, compare=close_on_row_scale)


@pytest.mark.parametrize("name", ["brief", "brief_d32", "brief_d128", "brief_alone", "brief_alone_d128", "one_way", "one_way_rt", "two_ways", "four_ways_d128",
                                  "ordinary_d32", "ordinary_d32_rt", "ordinary_d128_rt", "one_pass", "rows_resident"])
def test_non_finite_values_stay_with_their_user(name):
    """The users that own the call's first and last query rows get NaN everywhere; everyone else's results keep their bits.  (Lanes
    that stand for no row still multiply their dP by a weight of 0: it has to be the dP of a row of the same user.)"""
    case, _ = make(name)
    rows = np.diff(case.q_offsets)
    spoilt = [int(np.flatnonzero(rows)[0]), int(np.flatnonzero(rows)[-1])]
    q_keep, kv_keep = np.ones(case.total_q, bool), np.ones(case.total_kv, bool)
    for b in spoilt:
        q_keep[case.q_offsets[b]:case.q_offsets[b + 1]] = False
        kv_keep[case.kv_offsets[b]:case.kv_offsets[b + 1]] = False
    q_keep, kv_keep = torch.from_numpy(q_keep).to("cuda"), torch.from_numpy(kv_keep).to("cuda")
    results = []
    for value in (None, float("nan")):
        batch, dout = device_batch(case), to_torch(case.dout, "bf16")
        if value is not None:
            batch.q[~q_keep], batch.k[~kv_keep], batch.v[~kv_keep], dout[~q_keep] = value, value, value, value
        out, lse = batch.forward()
        dq, dk, dv = batch.backward(dout)
        results.append({"out": out[q_keep], "lse": lse[:, q_keep], "dq": dq[q_keep], "dk": dk[kv_keep], "dv": dv[kv_keep]})
    for key, clean in results[0].items():
        lost = int((results[1][key] != clean).sum())
        say(f"    {name} {key}: {lost} of {clean.numel()} elements of the other users changed")
        assert torch.isfinite(clean).all() and lost == 0, f"{key}: {lost} elements of other users changed"
