"""Nearest-neighbour staging and selection at their edges: rows staged by 1 to
64 lanes in one or several rounds (16 to 512 bytes, one to eight waves), score
terms summed while staging, and 4, 8 or 16 targets per selecting workgroup,
against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from _gpu_util import need_gpu

pytestmark = pytest.mark.gpu

CASES = [
    # T, M, D, configuration
    (70, 301, 16, "nt=1 wv=8 bt=2 tg=1 ch=3"), (70, 301, 32, "nt=2 wv=1 bt=8 tg=4 ch=9"),
    (33, 500, 48, "nt=1 wv=3 bt=2 tg=2 ch=5"), (33, 500, 80, "nt=1 wv=4 bt=1 tg=1 ch=2"),
    (45, 260, 144, "nt=2 wv=8 bt=2 tg=1 ch=4"), (45, 260, 144, "nt=5 wv=2 bt=8 tg=2 ch=8"),
    (20, 130, 400, "nt=1 wv=8 bt=1 tg=1 ch=3"), (20, 130, 512, "nt=2 wv=8 bt=2 tg=2 ch=2"),
    (20, 17, 512, "nt=1 wv=1 bt=1 tg=1 ch=1"), (2047, 40, 16, ""), (2050, 65, 48, "fw=1"), (4100, 33, 16, "fw=16"),
    (4097, 50, 64, "fw=2"),
]


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("T,M,D,cfg", CASES)
def test_exact(T, M, D, cfg, split):
    need_gpu()
    import torch
    from paper_0911_3456_amd import NNPlan
    rng = np.random.default_rng(T + M + D)
    t = rng.integers(0, 256, (T, D), dtype=np.uint8)
    n = rng.integers(0, 256, (M, D), dtype=np.uint8)
    n[M // 2] = n[1]                                  # a tie
    t[0] = n[1]
    t[1], n[M - 1] = 0, 255                           # the ends of the range
    plan = NNPlan(T, M, D)
    plan.set_config("%s split=%d" % (cfg, split))
    idx, dist = plan.search(torch.from_numpy(t).cuda(), torch.from_numpy(n).cuda())
    ri, rd = oracle.nearest(t, n)
    np.testing.assert_array_equal(idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(dist.cpu().numpy(), rd)
