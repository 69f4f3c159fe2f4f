"""GPU parity at inference shapes: forward only, a handful of requests, so the library splits the keys of every
(user, kv head) group over the waves of a workgroup, and over several workgroups where that pays, and merges the partial
softmax results.  Same float64 oracle, same tolerances (atol = rtol = 2e-2 for bf16) as the training shapes."""
import numpy as np
import pytest
import torch

from paper_2602_11235_amd import hta, inputs
from tests import test_gpu_parity_pointwise as pointwise
from tests.hta_testlib import check_case, compare_with_oracle, device_batch, form_of, host

pytestmark = pytest.mark.gpu
FULL, TARGET = inputs.LAYER_FULL, inputs.LAYER_TARGET


def is_split(case) -> bool:
    """Is the call small enough that its keys may be split over workgroups (the forward workspace has room for partial results)?"""
    b = device_batch(case)
    plain = 256 + 256 * ((4 * case.batch + 255) // 256)
    if case.rt_len is not None:
        plain += 256 * ((4 * case.total_q + 255) // 256)
    return b.fwd_workspace_bytes > plain


@pytest.mark.parametrize("name", ["I1", "I2", "I3", "I2_RT"])
def test_inference_workloads_forward(name):
    c = inputs.make_case(inputs.CONFIGS[name])
    assert is_split(c)
    check_case(c, with_bwd=False)


# Histories around the tile and block boundaries next to long ones: no history at all (no wave has a key, the own key alone),
# less than one tile, exactly two tiles, one key more than a tile.
EDGE_HIST = [2048, 0, 1, 63, 128, 65, 1000, 64]
EDGE_TGTS = [16, 5, 1, 33, 64, 2, 70, 0]


@pytest.mark.parametrize("layer", [TARGET, FULL])
@pytest.mark.parametrize("Hq,Hkv,d", [(8, 2, 64), (2, 2, 64), (3, 1, 64), (16, 2, 128), (4, 2, 32), (6, 1, 128)])
def test_split_forward_edge_cases(layer, Hq, Hkv, d):
    hist, tg = (EDGE_HIST, EDGE_TGTS) if layer == TARGET else ([600, 63, 0], [16, 33, 5])  # full layer: few row tiles
    c = inputs.make_case(inputs.custom_config(f"split_{Hq}_{Hkv}_{d}", layer, hist, tg, Hq, Hkv, d, seed=31))
    assert is_split(c)
    check_case(c, with_bwd=(layer == FULL))   # the backward pass reads the merged out / lse


@pytest.mark.parametrize("layer", [TARGET, FULL])
def test_split_forward_with_real_time_tokens(layer):
    c = inputs.make_case(inputs.custom_config("split_rt", layer, [1500, 0, 63, 700], [16, 5, 33, 2], 8, 2, 64, seed=32,
                                              rt_len=[70, 5, 0, 130]))
    assert is_split(c)
    check_case(c, with_bwd=False)


# A history long enough that splitting it over workgroups pays for the launch that merges the partial results, next to users whose
# keys end in the first split or before it.
LONG_HIST = [8192, 0, 1, 63, 4133]
LONG_RT = [70, 5, 0, 130, 300]
LONG_TGTS = [16, 5, 1, 33, 2]


def config_of_long(heads, with_rt):
    return inputs.custom_config("split_long", TARGET, LONG_HIST, LONG_TGTS, *heads, seed=35, rt_len=LONG_RT if with_rt else None)


@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("heads", [(8, 2, 64), (3, 1, 64), (16, 2, 128), (4, 2, 32)])
def test_keys_split_over_workgroups(heads, with_rt):
    c = inputs.make_case(config_of_long(heads, with_rt))
    assert is_split(c)
    check_case(c, with_bwd=False)


@pytest.mark.parametrize("layer", [TARGET, FULL])
@pytest.mark.parametrize("heads", [(8, 2, 64), (3, 1, 128)])
def test_few_requests_with_many_real_time_tokens(layer, heads):
    """Real-time segments at and around the length up to which their timestamps are searched in LDS (512), and at its copies'
    64-token pieces; with the backward pass, which goes by the same limits."""
    c = inputs.make_case(inputs.custom_config("many_rt", layer, [700, 0, 63, 130, 200, 64], [16, 5, 33, 2, 7, 1], *heads, seed=34,
                                              rt_len=[512, 513, 600, 511, 65, 64]))
    check_case(c, with_bwd=True)


# The work items that a launch for requests makes of the lengths: users without a row or a key anywhere among them, more users than a wave has
# lanes (which stand in a grid), more items than compute units, pieces of keys that grow until the items fit, and splits that the shorter users do not reach.
LISTS = {
    "many_users": (TARGET, np.resize([0, 1, 31, 700, 64, 0, 1500, 33], 130), np.resize([1, 0, 3, 2, 0, 5, 1], 130), (4, 1, 64)),
    "a_lane_more": (TARGET, np.resize([40, 300, 0], 65), np.resize([2, 0, 1, 3], 65), (8, 2, 32)),
    "three_waves_of_users": (TARGET, np.resize([90, 0, 260], 192), np.resize([1, 2, 0], 192), (2, 1, 128)),
    "pieces_grow": (TARGET, [6000, 300, 0, 4100, 2500, 65, 3300, 5000], [90, 30, 5, 70, 0, 64, 33, 50], (8, 2, 64)),
    "more_than_units": (TARGET, np.resize([1400, 900, 63, 2000], 20), np.resize([70, 33, 128, 0], 20), (16, 4, 64)),
    "two_row_blocks_d128": (TARGET, np.resize([1100, 0, 640, 33], 20), np.resize([64, 5, 100, 17], 20), (16, 2, 128)),
    "two_row_blocks_d128_in_pieces": (TARGET, [8192, 7000, 100, 8000], [80, 76, 3, 66], (16, 2, 128)),
    "two_row_blocks_d128_full": (FULL, [300, 200, 40], [20, 5, 17], (16, 2, 128)),
    "many_pieces": (TARGET, [16384, 200], [3, 2], (4, 1, 64)),
}


def config_of_list(name, with_rt, seed=36):
    layer, hist, targets, heads = LISTS[name]
    return inputs.custom_config(name, layer, hist, targets, *heads, seed=seed, rt_len=np.resize([40, 0, 7, 130, 1], len(hist)) if with_rt else None)


@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("name", LISTS)
def test_lists_of_items(name, with_rt):
    check_case(inputs.make_case(config_of_list(name, with_rt)), with_bwd=False)


@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("name", ["pieces_grow", "two_row_blocks_d128", "two_row_blocks_d128_in_pieces", "many_users"])
def test_lists_of_items_pointwise(name, with_rt):
    pointwise.check(inputs.make_case(config_of_list(name, with_rt, seed=37)))


# More users than a list has lanes: a list that takes two or three rounds of lanes where a grid would have more places than there are units,
# and a grid; one and two row blocks, keys in one piece and in several, users without a row or a key.  (form: in pieces, row blocks, grid)
MANY = {
    "list_of_two_rounds": (np.resize([40, 300, 0, 700], 100), np.resize([20, 0, 9, 33], 100), (8, 2, 64), (False, 1, 0)),
    "list_of_three_rounds": (np.resize([1500, 0, 640, 64], 170), np.resize([13, 0, 9, 8], 170), (8, 1, 128), (False, 1, 0)),
    "list_of_three_rounds_64_rows": (np.resize([1500, 1400], 190), np.resize([13, 8], 190), (8, 1, 64), (False, 2, 0)),
    "grid": (np.resize([300, 250, 0, 310], 300), np.resize([1, 0, 3], 300), (8, 1, 32), (False, 1, 1)),
    "grid_64_rows": (np.resize([1000, 900], 250), np.resize([16, 15], 250), (4, 1, 64), (False, 2, 1)),
    "grid_64_rows_d128": (np.resize([1000, 900], 225), np.resize([8, 7], 225), (8, 1, 128), (False, 2, 1)),
    "grid_in_pieces": (np.resize([8192, 0, 300, 5000, 7000], 66), np.resize([1, 2, 0, 3], 66), (8, 1, 64), (True, 1, 1)),
    "grid_in_pieces_d32": (np.resize([16384, 8000, 300, 12000], 66), np.resize([1, 2, 0, 3], 66), (8, 1, 32), (True, 1, 1)),
    "grid_in_pieces_d128": (np.resize([8192, 0, 300, 5000, 6000], 66), np.resize([1, 2, 0, 3], 66), (8, 1, 128), (True, 1, 1)),
}


@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("name", MANY)
def test_many_users(name, with_rt):
    hist, targets, heads, form = MANY[name]
    case = inputs.make_case(inputs.custom_config(name, TARGET, hist, targets, *heads, seed=41, rt_len=np.resize([40, 0, 7, 130, 1], len(hist)) if with_rt else None))
    taken = form_of(case.cfg, hta.CALL_FWD)
    assert (taken.kind > 1, taken.ways, taken.option) == form and taken.kind > 0
    check_case(case, with_bwd=False, users=sorted(set(range(0, len(hist), 7)) | {1, 63, 64, 65, len(hist) - 1}))


@pytest.mark.parametrize("users", [193, 197, 224])
@pytest.mark.parametrize("tiles", [2, 3, 4, 5])
def test_tiles_of_a_grid(tiles, users):
    """Users with all the tiles (of 8 rows) that the bounds allow next to users with one or none: every tile has one place."""
    targets = np.resize([1, 0, 2, 1, 1, 1, 0, 1, 1, 8 * tiles, 1, 1, 0, 1, 8 * tiles - 7, 1, 1], users)
    case = inputs.make_case(inputs.custom_config("tiles", TARGET, np.resize([300, 0, 250], users), targets, 4, 1, 64, seed=47))
    assert form_of(case.cfg, hta.CALL_FWD)[:3] == (1, 1, 1)
    check_case(case, with_bwd=False)


def with_bounds(batch: hta.Batch, factor: int, of_targets: int = 1) -> hta.Batch:
    """The same call with host bounds that far above its lengths, as a captured graph for requests of many sizes has them."""
    return hta.Batch(batch.q, batch.k, batch.v, batch.q_offsets, batch.kv_offsets, batch.hist_len, batch.n_targets, batch.max_hist * factor,
                     batch.max_targets * of_targets, batch.softmax_scale, batch.layer, batch.rt_len, batch.timestamps, batch.max_rt * factor)


@pytest.mark.parametrize("factor", [2, 16])
@pytest.mark.parametrize("with_rt", [False, True])
@pytest.mark.parametrize("name", ["pieces_grow", "more_than_units", "two_row_blocks_d128_in_pieces", "many_pieces", "many_users"])
def test_lists_of_items_with_bounds_above_the_lengths(name, with_rt, factor):
    case = inputs.make_case(config_of_list(name, with_rt, seed=39))
    out, lse = with_bounds(device_batch(case), factor, of_targets=factor).forward()
    compare_with_oracle(case, {"out": out, "lse": lse}, with_bwd=False)


def pieces_of_first_row(batch: hta.Batch) -> int:
    """Partial results of the call's first row, head 0, by what its logsumexps in the workspace say after a call.  (Behind counters and
    order, 512 bytes with up to 64 users: partial outputs [splits][total_q][Hq][d], logsumexps [splits][Hq][total_q], float32.)"""
    per_split = batch.total_q * batch.Hq * 4
    assert batch.batch <= 64 and batch.rt_len is None and per_split % 256 == 0
    splits = (batch.fwd_workspace_bytes - 512) // (per_split * (batch.head_dim + 1))
    batch.fwd_workspace.fill_(0xff)  # (NaN)
    batch.forward()
    lse = batch.fwd_workspace[512 + splits * per_split * batch.head_dim:].view(torch.float32)[:splits * per_split // 4]
    return int(lse.view(splits, -1)[:, 0].isfinite().sum())


@pytest.mark.parametrize("heads", [(8, 2, 64), (16, 2, 128), (4, 2, 32)])
def test_pieces_come_from_the_lengths(heads):
    """Keys are cut into as many pieces, or more, when the bounds are far above them.  (By the bounds alone it was one or two pieces.)"""
    case = inputs.make_case(inputs.custom_config("pieces", TARGET, [8192, 8000], [64, 64], *heads, seed=40))
    pieces = [pieces_of_first_row(b) for b in (device_batch(case), with_bounds(device_batch(case), 8))]
    assert 1 < pieces[0] <= pieces[1]


# keys in one piece and in several, one and two row blocks
@pytest.mark.parametrize("name,hist,targets,heads", [("one_piece", [700, 90], [20, 3], (8, 2, 64)), ("pieces", [8192, 300], [20, 3], (8, 2, 64)),
                                                     ("one_piece_64_rows_d128", [1100, 300, 640, 33] * 5, [64, 5, 100, 17] * 5, (16, 2, 128)),
                                                     ("pieces_64_rows_d128", [8192, 7000, 100, 8000], [64, 60, 3, 50], (16, 2, 128))])
def test_nan_shows(name, hist, targets, heads):
    """A NaN key reaches every row that sees it, in out and in lse, and no other: the own key of a candidate, and a key far back in a history."""
    case = inputs.make_case(inputs.custom_config(name, TARGET, hist, targets, *heads, seed=38))
    form, rows64 = form_of(case.cfg, hta.CALL_FWD), "64_rows" in name
    assert (form.kind > 1) == name.startswith("pieces") and form.kind > 0 and form.ways == (2 if rows64 else 1)
    r, nan = heads[0] // heads[1], float("nan")
    clean, clean_lse = device_batch(case).forward()
    for key, rows in ((hist[0] + 1, slice(1, 2)), (hist[0] * 7 // 8, slice(0, targets[0]))):
        batch = device_batch(case)
        batch.k[key, 0, 5] = nan
        out, lse = batch.forward()
        expected = torch.zeros(out.shape[:2], dtype=torch.bool, device="cuda")
        expected[rows, :r] = True
        assert torch.equal(out.isnan().all(dim=2), expected)
        assert torch.equal(out[~expected], clean[~expected])
        assert torch.equal(lse.isnan(), expected.T)
        assert torch.equal(lse[~expected.T], clean_lse[~expected.T])


def test_split_and_unsplit_forward_agree():
    """The same request alone (keys split over waves) and as one of 300 copies (not split): two different summation orders of
    the same softmax, equal up to the bf16 rounding of the output."""
    one = inputs.make_case(inputs.custom_config("one", TARGET, [1800], [40], 8, 2, 64, seed=33))
    many = inputs.take_users(one, [0] * 300)
    assert is_split(one) and not is_split(many)
    a_out, a_lse = device_batch(one).forward()
    b_out, b_lse = device_batch(many).forward()
    torch.cuda.synchronize()
    n = one.total_q
    assert np.allclose(host(a_out), host(b_out)[:n], rtol=2e-2, atol=2e-3)
    # (the row sums are formed from bf16-rounded weights, so lse carries ~1e-3 of rounding in either order)
    assert np.allclose(host(a_lse), host(b_lse)[:, :n], rtol=2e-3, atol=2e-3)
