"""Filter gradient with fp32 operands as three bf16 parts (algo=dws) against
the FP64 oracle, through the C ABI: bit for bit on integer-valued inputs over
tilings that reach its edges (ragged strips and segments, two rows per step,
several column blocks, uneven tile deals, filters past the bank, shifted
copies for channel counts that are not a multiple of 4); what fp32 arithmetic
gives for values that the parts cannot hold; and the tiling rule's choice
builds for every problem of a random sample."""
import numpy as np
import pytest

import oracle
import workloads as wl
from _gpu_util import host, need_gpu, to_dev

TOL = 1e-5

# (batch, H, W, D, N, fh, fw), configuration
CASES = [
    ((2, 41, 67, 8, 64, 9, 9), "rt=4 nw=8 ncb=2 rh=1 rw=64 rseg=8 np=10"),          # 41 column tiles over 16 waves
    ((2, 41, 67, 8, 64, 9, 9), "rt=2 nw=4 ncb=3 rh=2 rw=32 rseg=10 np=7"),          # segments left over
    ((1, 33, 41, 16, 40, 5, 4), "rt=3 nw=6 ncb=1 rh=2 rw=48 rseg=6 np=5"),          # 40 filters in 48
    ((1, 30, 37, 24, 100, 3, 3), "rt=4 nw=4 ncb=2 rh=1 rw=32 rseg=7 np=9"),         # 100 filters in 2 x 64
    ((2, 40, 50, 3, 10, 3, 4), "rt=1 nw=2 ncb=1 rh=2 rw=48 rseg=7 np=20"),          # four shifted copies
    ((2, 40, 50, 1, 20, 5, 5), "rt=2 nw=2 ncb=1 rh=1 rw=32 rseg=5 np=8"),
    ((1, 25, 90, 6, 17, 2, 5), "rt=2 nw=4 ncb=1 rh=2 rw=16 rseg=4 np=30"),          # two copies
    ((1, 9, 11, 5, 33, 9, 11), "rt=3 nw=8 ncb=2 rh=2 rw=16 rseg=2 np=1"),           # one output pixel
    ((3, 20, 21, 4, 1, 1, 1), "rt=1 nw=2 ncb=1 rh=2 rw=16 rseg=40 np=4"),           # more waves than tiles
]


def _dw(s, cfg, x, w, g):
    from paper_0911_3456_amd import Plan
    p = Plan(s.batch, s.H, s.W, s.D, s.N, s.fh, s.fw)
    if cfg:
        p.set_config("backward_w", "algo=dws " + cfg)
    xt, wt, gt = to_dev(x, w, g)
    a = host(p.backward(xt, wt, gt, need_dx=False)[1])
    b = host(p.backward(xt, wt, gt, need_dx=False)[1])
    np.testing.assert_array_equal(a, b)           # the same bits every time
    return a


def test_configurations_are_valid():
    from paper_0911_3456_amd import FbcorrError, codegen, make_desc
    for sh, cfg in CASES:
        codegen(make_desc(*sh), "backward_w", "algo=dws " + cfg)
    d = make_desc(2, 41, 67, 8, 64, 9, 9)
    good = "algo=dws rt=2 nw=4 ncb=3 rh=2 rw=32 rseg=10 np=7"
    for bad in ["rt=5", "rw=24", "rh=1 rw=48", "np=0", "nw=17", "rt=4 nw=2 ncb=1", "tpb=3"]:
        with pytest.raises(FbcorrError):
            codegen(d, "backward_w", good + " " + bad)


def test_rule_builds_every_problem():
    from paper_0911_3456_amd import FbcorrError, codegen, make_desc
    rng = np.random.default_rng(4)
    seen = set()
    for _ in range(150):
        fh, fw = (int(v) for v in rng.integers(1, 14, 2))
        H, W = fh + int(2 ** rng.uniform(0, 9)) - 1, fw + int(2 ** rng.uniform(0, 9)) - 1
        d = make_desc(int(rng.integers(1, 9)), H, W, int(2 ** rng.uniform(0, 7)), int(2 ** rng.uniform(0, 8)), fh, fw)
        try:
            codegen(d, "backward_w", "algo=dw")
        except FbcorrError:                       # more filter taps than the plain kernel holds
            with pytest.raises(FbcorrError):
                codegen(d, "backward_w", None)
            continue
        seen.add("-DFB_RSEG" in codegen(d, "backward_w", None)[1])
    assert True in seen


@pytest.mark.gpu
@pytest.mark.parametrize("shape,cfg", CASES + [((2, 45, 77, 12, 30, 5, 3), "")])
def test_integer_exact(shape, cfg):
    need_gpu()
    s = wl.Shape(*shape)
    x, w, rng = wl.draw_integer(s, seed=800 + sum(shape), xmax=3, wmax=2)
    g = rng.integers(-3, 4, size=(s.batch, s.Ho, s.Wo, s.N)).astype(np.float32)
    _, rw = oracle.backward(x, w, g)
    np.testing.assert_array_equal(_dw(s, cfg, x, w, g), rw.astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,cfg", [CASES[0], CASES[4]])
def test_random_within_fp32_bound(shape, cfg):
    need_gpu()
    s = wl.Shape(*shape)
    x, w, rng = wl.draw_single(s, seed=900 + sum(shape))
    g = wl.draw_grad(s, rng)
    _, rw = oracle.backward(x, w, g)
    _, sw = oracle.backward_scales(x, w, g)
    assert oracle.normalised_error(_dw(s, cfg, x, w, g), rw, sw)[0] <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["inf", "nan", "lowest", "tiny", "huge", "tiny_gradient"])
def test_values_outside_the_parts(name):
    need_gpu()
    s = wl.Shape(2, 30, 40, 8, 24, 5, 3)
    x, w, rng = wl.draw_single(s, seed=32)
    g = wl.draw_grad(s, rng)
    if name == "inf":
        x[1, 10, 10, 1] = np.inf
    elif name == "nan":
        g[0, 20, 10, 1] = np.nan
    elif name == "lowest":
        x[0, 12, 12, 2] = np.finfo(np.float32).min
        g *= np.float32(0.01)
    elif name == "tiny":
        x[0] *= np.float32(1e-34)
    elif name == "huge":
        x *= np.float32(1e25)
    elif name == "tiny_gradient":
        g[..., 3] *= np.float32(1e-33)
    dw = _dw(s, "rt=2 nw=4 ncb=1 rh=1 rw=32 rseg=6 np=8", x, w, g).astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref, scl = np.zeros(w.shape), np.zeros(w.shape)
        for u in range(s.fh):
            for v in range(s.fw):
                a = g[..., :, None].astype(np.float64) * x[:, u:u + s.Ho, v:v + s.Wo, None, :].astype(np.float64)
                ref[:, u, v] = a.sum(axis=(0, 1, 2))
                scl[:, u, v] = np.abs(a).sum(axis=(0, 1, 2))
    np.testing.assert_array_equal(np.isnan(dw), np.isnan(ref))
    inf = np.isinf(ref)
    np.testing.assert_array_equal(dw[inf], ref[inf])
    fin = np.isfinite(ref)
    assert (np.abs(dw[fin] - ref[fin]) <= TOL * scl[fin]).all()
