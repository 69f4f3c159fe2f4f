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
