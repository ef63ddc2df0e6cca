"""The timer of a batched plan covers every kernel of a launch: with banks
that take longer to pack than the few output pixels take to compute, its
total is the launches' time, not a part of it."""
import pytest

from _gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def test_timer_includes_the_packing():
    need_gpu()
    import torch
    from paper_0911_3456_amd import BatchedPlan
    shapes = [(12, 12, 32, 512, 9, 9)] * 12          # 12 banks of 5 MB, 16 output pixels each
    plan = BatchedPlan(shapes)
    assert "sp=1" in plan.describe()
    xs = [torch.rand(s[:3], device="cuda") for s in shapes]
    ws = [torch.randn((s[3], s[4], s[5], s[2]), device="cuda") for s in shapes]
    plan.forward(xs, ws)
    torch.cuda.synchronize()
    n = 100
    plan.read_timing(reset=True)
    plan.enable_timing(True)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(n):
        plan.launch()
    b.record()
    torch.cuda.synchronize()
    plan.enable_timing(False)
    ms, calls = plan.read_timing()
    total = a.elapsed_time(b)
    print("timer %.3f ms of %.3f ms" % (ms, total))
    assert calls == n and 0.8 * total <= ms <= 1.05 * total
