"""fp32 operands as three bf16 parts on the matrix cores (rgemm with sp=1)
against the FP64 oracle, through the C ABI: the forward correlation and the
input gradient.

* integer-valued inputs (exact partial sums): bit for bit, over tilings that
  reach every layout of the staged tile (planes of cells, rows of 4, 12 and 24
  channels, odd channel counts with a column shift), steps that straddle
  filter rows, a padded last step, several channel chunks and masked stores;
* values that the parts cannot hold (infinities, NaNs, magnitudes near the
  ends of the fp32 range) give what fp32 arithmetic gives: the same non-finite
  outputs as the fp64 sum, the finite ones within the fp32 bound;
* the rule that picks tilings: every problem of a random sample builds.
"""
import numpy as np
import pytest

import oracle
import workloads as wl
from _gpu_util import forward_error, host, need_gpu, to_dev

FP32_TOL = 1e-5

# (batch, H, W, D, N, fh, fw), configuration
CASES = [
    ((2, 45, 77, 8, 64, 9, 9), "mf=32 kc=8 mr=2 mt=2 nt=2 wm=2 wn=1 pf=2 ste=1"),      # 81 cells: padded last step
    ((2, 45, 77, 8, 64, 9, 9), "mf=16 kc=8 mr=1 mt=4 nt=2 wm=4 wn=2 pf=2 ste=1 nts=1"),
    ((1, 33, 41, 16, 40, 5, 4), "mf=16 kc=16 mr=4 mt=4 nt=1 wm=2 wn=1 pf=2 ste=1"),     # masked 16-byte stores
    ((1, 40, 39, 48, 24, 3, 3), "mf=32 kc=16 mr=4 mt=1 nt=1 wm=4 wn=1 pf=2"),           # three chunks
    ((1, 40, 39, 48, 24, 3, 3), "mf=16 kc=24 mr=2 mt=2 nt=2 wm=2 wn=1 pf=2"),           # rows of 24 channels
    ((2, 30, 33, 12, 20, 5, 3), "mf=16 kc=12 mr=1 mt=2 nt=2 wm=2 wn=1 pf=2"),           # rows of 12 channels
    ((1, 37, 50, 3, 32, 7, 7), "mf=16 kc=4 mr=1 mt=4 nt=2 wm=2 wn=1 pf=2 ste=1"),       # 3 channels padded to 4
    ((1, 37, 50, 3, 20, 7, 5), "mf=16 s=4 kc=3 mr=2 mt=2 nt=2 wm=2 wn=1 pf=2"),         # 3 channels as they are
    ((2, 41, 39, 1, 10, 11, 11), "mf=32 s=4 kc=1 mr=2 mt=1 nt=2 wm=2 wn=1 pf=2"),       # one channel
    ((1, 30, 47, 6, 9, 2, 5), "mf=16 s=2 kc=6 mr=4 mt=1 nt=2 wm=2 wn=1 pf=2"),
    ((1, 30, 47, 16, 7, 3, 3), "mf=16 s=2 kc=16 mr=1 mt=2 nt=1 wm=2 wn=1 pf=2"),        # shifted, planes by phase
    ((1, 9, 11, 5, 33, 9, 11), "mf=16 kc=8 mr=1 mt=1 nt=3 wm=2 wn=1 pf=2"),             # one output pixel
    ((3, 20, 21, 1, 1, 1, 1), "mf=16 s=4 kc=1 mr=1 mt=1 nt=1 wm=2 wn=1 pf=1"),          # a single step
]


def _plan(s, role, cfg):
    from paper_0911_3456_amd import Plan
    p = Plan(s.batch, s.H, s.W, s.D, s.N, s.fh, s.fw)
    p.set_config(role, cfg)
    return p


def test_configurations_are_valid():
    from paper_0911_3456_amd import codegen, make_desc
    for sh, cfg in CASES:
        _, o = codegen(make_desc(*sh), "forward", "algo=rgemm sp=1 " + cfg)
        assert "-DFB_DT=3" in o


def test_rule_builds_every_problem():
    """The tiling rule's choice is valid for every problem (the generator
    checks registers, LDS and divisibility) in every role and precision."""
    from paper_0911_3456_amd import codegen, make_desc
    rng = np.random.default_rng(3)
    seen = set()
    for _ in range(150):
        fh, fw = (int(v) for v in rng.integers(1, 14, 2))
        b = int(rng.integers(1, 9))
        H, W = fh + int(2 ** rng.uniform(0, 9)) - 1, fw + int(2 ** rng.uniform(0, 9)) - 1
        D, N = int(2 ** rng.uniform(0, 7)), int(2 ** rng.uniform(0, 8))
        for prec in ("fp32", "bf16", "fp16"):
            _, o = codegen(make_desc(b, H, W, D, N, fh, fw, precision=prec), "forward", None)
            seen.add((prec, "fbcorr_fwd_rgemm" in o, "-DFB_DT=3" in o))
        _, o = codegen(make_desc(b, H, W, D, N, fh, fw), "backward_x", None)
        seen.add(("dx", "fbcorr_dx_rgemm" in o, "-DFB_DT=3" in o))
    # both sides of the rule are reached
    assert {("fp32", True, True), ("fp32", False, False), ("bf16", True, False), ("fp16", True, False),
            ("dx", True, True)} <= seen


@pytest.mark.gpu
@pytest.mark.parametrize("shape,cfg", CASES)
def test_forward_integer_exact(shape, cfg):
    need_gpu()
    s = wl.Shape(*shape)
    x, w, _ = wl.draw_integer(s, seed=500 + sum(shape))
    y = host(_plan(s, "forward", "algo=rgemm sp=1 " + cfg).forward(*to_dev(x, w)))
    np.testing.assert_array_equal(y, oracle.forward(x, w).astype(np.float32))


# the input gradient contracts over N and has D outputs
DX_CASES = [
    ((2, 41, 67, 16, 64, 7, 7), "mf=16 kc=32 mr=1 mt=4 nt=1 wm=4 wn=1 pf=2 ste=1"),
    ((2, 41, 67, 8, 64, 9, 9), "mf=16 s=2 kc=16 mr=2 mt=2 nt=1 wm=4 wn=1 pf=2"),
    ((1, 30, 33, 3, 20, 5, 4), "mf=16 s=4 kc=20 mr=2 mt=1 nt=1 wm=2 wn=1 pf=2"),
    ((1, 25, 31, 24, 10, 3, 3), "mf=32 s=2 kc=10 mr=2 mt=1 nt=2 wm=2 wn=1 pf=2"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,cfg", DX_CASES)
def test_dx_integer_exact(shape, cfg):
    need_gpu()
    s = wl.Shape(*shape)
    x, w, rng = wl.draw_integer(s, seed=600 + sum(shape), xmax=2, wmax=2)
    g = rng.integers(-2, 3, size=(s.batch, s.Ho, s.Wo, s.N)).astype(np.float32)
    xt, wt, gt = to_dev(x, w, g)
    dx, _ = _plan(s, "backward_x", "algo=rgemm sp=1 " + cfg).backward(xt, wt, gt, need_dw=False)
    rx, _ = oracle.backward(x, w, g, want_dw=False)
    np.testing.assert_array_equal(host(dx), rx.astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,cfg", [CASES[1], CASES[6], CASES[8]])
def test_random_error_below_fp32_instructions(shape, cfg):
    """No worse than the same tiles on fp32 matrix instructions."""
    need_gpu()
    s = wl.Shape(*shape)
    x, w, _ = wl.draw_single(s, seed=700 + sum(shape))
    y_ref, xt, wt = oracle.forward(x, w), *to_dev(x, w)
    e, mean, _ = forward_error(host(_plan(s, "forward", "algo=rgemm sp=1 " + cfg).forward(xt, wt)), x, w, y_ref)
    e0, mean0, _ = forward_error(host(_plan(s, "forward", "algo=igemm").forward(xt, wt)), x, w, y_ref)
    assert e <= FP32_TOL and mean <= mean0, (e, e0, mean, mean0)


def _special(name, x, w, rng):
    if name == "inf":
        x[0, 10, 10, 1] = np.inf
    elif name == "nan":
        x[0, 20, 10, 1] = np.nan
    elif name == "lowest":
        x[0, 12, 12, 2] = np.finfo(np.float32).min
        w *= np.float32(0.25)
    elif name == "tiny":
        x[0, 5:20, 5:20] *= np.float32(1e-33)
    elif name == "huge":
        x *= np.float32(1e33)
    elif name == "filter_inf":
        w[3, 1, 1, 1] = -np.inf
    elif name == "filter_tiny":
        w[5] *= np.float32(1e-30)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["inf", "nan", "lowest", "tiny", "huge", "filter_inf", "filter_tiny"])
@pytest.mark.parametrize("cfg", ["mf=32 kc=8 mr=2 mt=1 nt=1 wm=2 wn=1 pf=2", "mf=16 s=2 kc=8 mr=1 mt=2 nt=3 wm=2 wn=1 pf=2"])
def test_values_outside_the_parts(name, cfg):
    need_gpu()
    s = wl.Shape(1, 40, 50, 8, 24, 5, 3)
    x, w, rng = wl.draw_single(s, seed=31)
    _special(name, x, w, rng)
    y = host(_plan(s, "forward", "algo=rgemm sp=1 " + cfg).forward(*to_dev(x, w))).astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref, scl = np.zeros(y.shape), np.zeros(y.shape)
        for u in range(s.fh):
            for v in range(s.fw):
                a = x[:, u:u + s.Ho, v:v + s.Wo, :, None].astype(np.float64) * w[:, u, v].T.astype(np.float64)
                ref += a.sum(axis=3)
                scl += np.abs(a).sum(axis=3)
    np.testing.assert_array_equal(np.isnan(y), np.isnan(ref))
    inf = np.isinf(ref)
    np.testing.assert_array_equal(y[inf], ref[inf])
    fin = np.isfinite(ref)
    err = np.abs(y[fin] - ref[fin])
    assert (err <= FP32_TOL * scl[fin]).all(), np.nanmax(err / np.maximum(scl[fin], 1e-300))


def test_large_banks_stay_within_the_static_scratch():
    """A forward pass that fits the allocation-free entry point's scratch
    with the plain kernel is not moved to one that does not."""
    from paper_0911_3456_amd import codegen, make_desc
    _, o = codegen(make_desc(1, 40, 40, 64, 1024, 13, 13), "forward", None)       # 66 MB as bf16 parts
    assert "-DFB_DT=0" in o
    _, o = codegen(make_desc(1, 40, 40, 64, 256, 7, 7), "forward", None)
    assert "-DFB_DT=3" in o
