"""A batch of more tiles than one launch can have workgroups (2^32 threads):
nine images of 2e9 pixels that share their buffers, but for the last one's
output."""
import pytest

from _gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def test_more_tiles_than_a_launch():
    need_gpu()
    import torch
    from paper_0911_3456_amd import BatchedPlan
    if torch.cuda.get_device_properties(0).total_memory < 100 << 30:
        pytest.skip("needs 50 GB of device memory")
    side = 44700
    plan = BatchedPlan([(side, side, 1, 1, 1, 1)] * 9)
    items = int(plan.describe().split("items=")[1].split()[0])
    assert items * 256 > 1 << 32
    x = torch.empty((side, side, 1), device="cuda").uniform_(-1, 1)
    w = torch.full((1, 1, 1, 1), 2.0, device="cuda")
    y, last = torch.zeros_like(x), torch.zeros_like(x)
    print("launch", items, flush=True)
    plan.forward([x] * 9, [w] * 9, [y] * 8 + [last])
    torch.cuda.synchronize()
    x.mul_(2)
    assert torch.equal(y, x) and torch.equal(last, x)
