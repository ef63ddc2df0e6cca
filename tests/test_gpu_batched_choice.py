"""Which variants a batched plan takes: three-part products where the images
have output pixels enough to pay for packing their banks, fp32 instructions
where many banks meet few pixels; both exact on integers."""
import numpy as np
import pytest

import oracle
import workloads as wl
from _gpu_util import host, need_gpu, to_dev

pytestmark = pytest.mark.gpu


# (images, D, N, filter side, output side), three parts?
BATCHES = [
    ((256, 64, 256, 3, 4), False),
    ((256, 64, 256, 3, 23), True),
    ((256, 16, 64, 5, 6), False),
    ((32, 16, 64, 5, 6), True),           # few workgroups: their own length counts
    ((48, 32, 512, 9, 4), False),
    ((48, 32, 512, 9, 23), True),
]


@pytest.mark.parametrize("batch,parts", BATCHES)
def test_choice(batch, parts):
    need_gpu()
    from paper_0911_3456_amd import BatchedPlan
    n, D, N, f, o = batch
    plan = BatchedPlan([(f + o - 1, f + o - 1, D, N, f, f)] * n)
    assert ("sp=1" in plan.describe()) == parts
    if n * N * f * f * D > 1e7:
        return
    rng = np.random.default_rng(n)
    xs = [rng.integers(-4, 5, (f + o - 1, f + o - 1, D)).astype(np.float32) for _ in range(n)]
    ws = [rng.integers(-4, 5, (N, f, f, D)).astype(np.float32) for _ in range(n)]
    ys = plan.forward(list(to_dev(*xs)), list(to_dev(*ws)))
    for k in (0, n // 2, n - 1):
        np.testing.assert_array_equal(host(ys[k]), oracle.forward(xs[k][None], ws[k])[0].astype(np.float32))


def test_choice_is_for_the_whole_batch():
    """Many keys of one image each fill the chip together: none of them
    counts on its own length."""
    need_gpu()
    from paper_0911_3456_amd import BatchedPlan
    shapes = [(8, 8, 16, 48 + 2 * k, 5, 5) for k in range(4)] * 64
    assert "sp=1" not in BatchedPlan(shapes).describe()
    assert "sp=1" in BatchedPlan([(120, 120, 16, 48 + 2 * k, 5, 5) for k in range(4)] * 16).describe()


def test_workload_keeps_its_parts():
    need_gpu()
    from paper_0911_3456_amd import BatchedPlan
    shapes, _ = wl.draw_batched_list()
    plan = BatchedPlan([(s.H, s.W, s.D, s.N, s.fh, s.fw) for s in shapes])
    assert "algo=igemm" not in plan.describe()


def test_single_pixel_windows():
    need_gpu()
    from paper_0911_3456_amd import BatchedPlan
    for D, parts in ((32, True), (64, False), (33, False)):
        assert ("sp=1" in BatchedPlan([(150, 150, D, 60, 1, 1)] * 32).describe()) == parts
