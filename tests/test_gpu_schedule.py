"""The order that the device gives a batch's users in: by decreasing work, ties by index, every user once; and, from the same launch,
the number of leading keys that each row sees with real-time tokens."""
import numpy as np
import pytest
import torch

from paper_2602_11235_amd import inputs
from tests.hta_testlib import device_batch, say, to_torch

pytestmark = pytest.mark.gpu
COUNTERS = 64  # int32 words in front of the order (QUEUE_WORDS)


@pytest.mark.parametrize("layer", [inputs.LAYER_FULL, inputs.LAYER_TARGET])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 255, 256, 257, 1000, 4096])   # 16 users to a workgroup, 256 threads; the largest
def test_order_of_the_users(layer, n):
    rng = np.random.RandomState(n)
    unit = max(4, 12000 // n)   # enough rows that the backward orders its users, however few
    hist, targets = rng.randint(0, 12, n) * unit, rng.randint(0, 4, n) * unit   # many ties, users without keys or rows
    hist[0], targets[0] = 5 * unit, 3 * unit
    rt = rng.randint(0, 3, n) if n % 2 else None
    if rt is not None:
        rt[0] = 2   # (none at all would be a call without them)
    say(f"  schedule layer={layer} n={n}")
    case = inputs.make_case(inputs.custom_config("order", layer, hist, targets, 4, 2, 32, seed=3, rt_len=rt))
    batch = device_batch(case)
    batch.forward()
    batch.prepare_backward()
    batch.workspace.fill_(0x7f)
    batch.backward(to_torch(case.dout, "bf16"))
    torch.cuda.synchronize()
    keys = hist + (0 if rt is None else rt)
    cost = (keys + targets if layer == inputs.LAYER_FULL else targets) * keys
    first = COUNTERS + (0 if rt is None else (case.total_q * 4 + 255) // 256 * 64)   # behind the rows' limits
    order = batch.workspace.view(torch.int32)[first:first + n].cpu().numpy()
    assert np.array_equal(order, np.argsort(-cost, kind="stable"))
    if rt is not None:
        lim = []
        for b, first_key in enumerate(case.kv_offsets[:-1]):
            ts = case.timestamps[first_key:case.kv_offsets[b + 1]]
            rows = ts if layer == inputs.LAYER_FULL else ts[keys[b]:]
            lim.append(hist[b] + np.searchsorted(ts[hist[b]:keys[b]], rows, side="left"))
        got = batch.workspace.view(torch.int32)[:case.total_q].cpu().numpy()
        assert np.array_equal(got, np.concatenate(lim))


@pytest.mark.parametrize("name,layer,users,hist,targets,heads", [
    ("one round, one pass", inputs.LAYER_TARGET, 250, 600, 64, (8, 2, 64)),      # 504 ids, room for 512 workgroups
    ("rounds, one pass", inputs.LAYER_TARGET, 1000, 150, 64, (8, 2, 64)),        # 2000 ids
    ("rounds, dK/dV", inputs.LAYER_FULL, 400, 700, 20, (4, 2, 32)),              # 4800 ids, mostly of one block of 128 keys
])
def test_workgroups_leave_an_exhausted_queue_without_counting_it_up(name, layer, users, hist, targets, heads):
    """The counters of the work queue after a call: what was taken behind the first round, one failing take per workgroup at its own
    list, and a few that lost a race at another one's.  (Counting up all eight lists before leaving: 8 per workgroup.)"""
    rng = np.random.RandomState(users)
    hist_len = np.full(users, hist) if layer == inputs.LAYER_TARGET else rng.randint(hist // 2, hist + 1, users)
    hist_len[0] = hist
    say(f"  queue {name}")
    case = inputs.make_case(inputs.custom_config("queue", layer, hist_len, np.full(users, targets), *heads, seed=4))
    batch = device_batch(case)
    batch.forward()
    batch.backward(to_torch(case.dout, "bf16"))
    torch.cuda.synchronize()
    counters = batch.workspace.view(torch.int32)[:COUNTERS].cpu().numpy()
    blocks = 1 if layer == inputs.LAYER_TARGET else -(-hist // 128)
    ids = -(-users * heads[1] // 8) * 8 * blocks
    units = torch.cuda.get_device_properties(0).multi_processor_count
    say(f"    {ids} ids, counters {counters[:8]}, {units} compute units")
    if name.startswith("one round"):
        assert not counters.any()
    else:
        assert 0 < counters.sum() < ids + 2 * units   # (512 or more workgroups: with 8 each it would be ids + 16 units)
    assert not counters[8:].any()
