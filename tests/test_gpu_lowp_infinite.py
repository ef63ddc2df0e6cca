"""Infinities and NaNs in 16-bit forwards reach the outputs whose windows hold
them and no others: not through the zero weights that fill a last step, a
row's last cell or a shifted column.  Against fp64 sums of the rounded
operands, default configurations."""
import numpy as np
import pytest

import oracle
from _gpu_util import host, need_gpu, to_dev

pytestmark = pytest.mark.gpu

# (batch, H, W, D, N, fh, fw)
SHAPES = [
    (1, 30, 37, 8, 40, 5, 3),          # 15 cells: a padded last step
    (2, 33, 41, 16, 64, 3, 3),         # 18 cells: padded in steps of 4
    (1, 40, 45, 4, 48, 3, 5),          # rows of 20 values in cells of 8
    (1, 38, 47, 12, 33, 2, 3),         # rows of 36
    (1, 60, 64, 3, 40, 7, 7),          # 3 channels
    (1, 70, 80, 1, 32, 5, 9),          # one channel: shifted columns
    (1, 90, 100, 16, 8, 4, 4),         # a narrow bank: shifted columns
]
CFGS = [None, "algo=rgemm mf=16 kc=8 mr=1 mt=2 nt=1 wm=2 wn=1 pf=2",
        "algo=rgemm mf=16 s=4 kc=8 mr=2 mt=2 nt=2 wm=2 wn=1 pf=2"]


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("cfg", CFGS)
@pytest.mark.parametrize("shape", SHAPES)
def test_where_infinities_go(shape, cfg, prec):
    need_gpu()
    from paper_0911_3456_amd import Plan
    B, H, W, D, N, fh, fw = shape
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal((B, H, W, D)).astype(np.float32)
    w = (rng.uniform(0.1, 1, (N, fh, fw, D)) * rng.choice([-1, 1], (N, fh, fw, D))).astype(np.float32)
    for k in range(4):                 # apart, so that windows hold one or none
        x[0, 4 + 9 * (k // 2), 5 + 16 * (k % 2), k % D] = (np.inf, -np.inf, np.nan, np.inf)[k]
    p = Plan(*shape, precision=prec)
    if cfg:
        p.set_config("forward", cfg)
    y = host(p.forward(*to_dev(x, w))).astype(np.float64)
    rnd = oracle.round_to_bf16 if prec == "bf16" else oracle.round_to_fp16
    sc = oracle.filter_pow2_scales(w)[:, None, None, None]
    fin = np.isfinite(x)
    xr = np.where(fin, rnd(np.where(fin, x, 0).astype(np.float32)), x).astype(np.float64)
    wr = rnd((w * sc).astype(np.float32)).astype(np.float64) / sc
    ho, wo = H - fh + 1, W - fw + 1
    ref, scl = np.zeros(y.shape), np.zeros(y.shape)
    with np.errstate(invalid="ignore"):
        for u in range(fh):
            for v in range(fw):
                a = xr[:, u:u + ho, v:v + wo, :, None] * wr[:, u, v].T
                ref += a.sum(axis=3)
                scl += np.abs(a).sum(axis=3)
    np.testing.assert_array_equal(np.isnan(y), np.isnan(ref))
    np.testing.assert_array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    assert np.isinf(ref).any() and np.isnan(ref).any() and (np.abs(y[ok] - ref[ok]) <= 1e-5 * scl[ok]).all()
