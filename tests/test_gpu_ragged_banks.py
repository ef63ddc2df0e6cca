"""Ragged banks: stores through LDS of a column block that the bank does not
fill, exact on integers."""
import numpy as np
import pytest

import oracle
import workloads as wl
from _gpu_util import host, need_gpu, to_dev


def test_streaming_stores_are_whole_pieces():
    from paper_0911_3456_amd import codegen, make_desc
    for N, nts in ((60, False), (64, True), (100, False), (48, True)):
        _, o = codegen(make_desc(4, 277, 277, 16, N, 5, 5), "forward", None)
        assert ("-DFB_NTS=1" in o) == nts


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("N,cfg", [
    (60, "mf=32 mt=1 nt=2 wm=2 wn=1"),            # one block of 64 columns
    (60, "mf=16 mt=2 nt=1 wm=2 wn=2 nts=1"),      # two of 32, the last with 28
    (100, "mf=32 mt=1 nt=1 wm=1 wn=3"),           # 96 and 4: waves without a column
    (4, "mf=16 mt=2 nt=2 wm=4 wn=1"),             # one vector a pixel
    (36, "mf=16 mt=1 nt=3 wm=2 wn=1"),            # 48 columns
])
def test_ragged_blocks_store_exactly(N, cfg, prec):
    need_gpu()
    from paper_0911_3456_amd import Plan
    s = wl.Shape(2, 37, 45, 8, N, 3, 3)
    x, w, _ = wl.draw_integer(s, seed=90 + N)
    p = Plan(s.batch, s.H, s.W, s.D, s.N, s.fh, s.fw, precision=prec)
    p.set_config("forward", "algo=rgemm kc=8 mr=2 pf=2 ste=1 " + ("sp=1 " if prec == "fp32" else "") + cfg)
    import torch
    xt, wt = to_dev(x, w)
    guard = torch.full((p.y_shape[0] * p.y_shape[1] * p.y_shape[2] * N + 256,), 7.0, device="cuda")
    y = guard[:-256].view(p.y_shape)              # nothing is written past the last pixel
    p.forward(xt, wt, y)
    np.testing.assert_array_equal(host(y), oracle.forward(x, w).astype(np.float32))
    assert float(host(guard[-256:]).min()) == 7.0 == float(host(guard[-256:]).max())
