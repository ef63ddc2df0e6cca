"""Batched launches whose variants hold fp32 operands as three bf16 parts:
bit for bit on integer-valued inputs over keys that reach the tilings' edges
(column shifts, channels that are not a multiple of 4, filters past the last
column block, one-pixel outputs), beside keys that stay with fp32
instructions; the bits of a single plan of the same configuration, also for
values that the parts cannot hold; and new contents, of images and banks, at
every replay of a graph."""
import numpy as np
import pytest

import oracle
import workloads as wl
from _gpu_util import host, need_gpu, to_dev

KEYS = [wl.Shape(1, 40, 61, 4, 5, 7, 3), wl.Shape(1, 33, 45, 3, 33, 5, 5), wl.Shape(1, 17, 90, 32, 100, 3, 3),
        wl.Shape(1, 51, 23, 10, 17, 4, 6), wl.Shape(1, 9, 9, 6, 130, 9, 9), wl.Shape(1, 30, 30, 1, 16, 3, 3),
        wl.Shape(1, 64, 9, 100, 40, 2, 9), wl.Shape(1, 25, 26, 3, 33, 5, 5)]


def _plan(shapes=KEYS):
    from paper_0911_3456_amd import BatchedPlan
    return BatchedPlan([(s.H, s.W, s.D, s.N, s.fh, s.fw) for s in shapes])


def _variants(plan):
    out = {}
    for part in plan.describe().split(" | ")[1:]:
        head, cfg = part.split(" algo=")
        t = dict(x.split("=") for x in head.split()[1:])
        out[tuple(int(t[k]) for k in ("fh", "fw", "D", "N"))] = "algo=" + cfg
    return out


def test_keys_compile():
    from paper_0911_3456_amd import compile_check_batched, make_desc
    assert compile_check_batched([make_desc(1, s.H, s.W, s.D, s.N, s.fh, s.fw) for s in KEYS]) > 0


@pytest.mark.gpu
def test_integer_exact_and_variants():
    need_gpu()
    rng = np.random.default_rng(61)
    xs = [rng.integers(-4, 5, size=(s.H, s.W, s.D)).astype(np.float32) for s in KEYS]
    fs = [rng.integers(-4, 5, size=(s.N, s.fh, s.fw, s.D)).astype(np.float32) for s in KEYS]
    plan = _plan()
    v = _variants(plan)
    assert "algo=igemm" in v[(3, 3, 1, 16)]           # nine taps of one channel: fp32 instructions
    assert all("sp=1" in c for k, c in v.items() if k != (3, 3, 1, 16)), v
    ys = plan.output_buffers()
    for y in ys:
        y.fill_(float("nan"))
    plan.forward(to_dev(*xs), to_dev(*fs), ys)
    for y, x, f in zip(ys, xs, fs):
        np.testing.assert_array_equal(host(y), oracle.forward(x, f).astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("plant", ["none", "large", "inf", "bank"])
def test_bits_of_a_single_plan(plant):
    need_gpu()
    from paper_0911_3456_amd import Plan
    rng = np.random.default_rng(62)
    xs = [rng.standard_normal((s.H, s.W, s.D)).astype(np.float32) for s in KEYS]
    fs = [rng.standard_normal((s.N, s.fh, s.fw, s.D)).astype(np.float32) for s in KEYS]
    for x, f in zip(xs, fs):
        if plant == "large":
            x[x.shape[0] // 2, 3, 0] = np.float32(2.0 ** 110)
        elif plant == "inf":
            x[2, x.shape[1] // 2, 0] = np.inf
        elif plant == "bank":
            f[1, 0, 0, 0] = np.nan
    plan = _plan()
    v = _variants(plan)
    ys = plan.forward(to_dev(*xs), to_dev(*fs))
    for s, x, f, y in zip(KEYS, xs, fs, ys):
        p = Plan(1, s.H, s.W, s.D, s.N, s.fh, s.fw)
        p.set_config("forward", v[(s.fh, s.fw, s.D, s.N)])
        xt, ft = to_dev(x[None], f)
        np.testing.assert_array_equal(host(y), host(p.forward(xt, ft))[0])


@pytest.mark.gpu
def test_replays_see_new_images_and_banks():
    need_gpu()
    import torch
    rng = np.random.default_rng(63)
    plan = _plan()
    xd = [torch.zeros((s.H, s.W, s.D), device="cuda") for s in KEYS]
    fd = [torch.zeros((s.N, s.fh, s.fw, s.D), device="cuda") for s in KEYS]
    ys = plan.output_buffers()
    plan.set_pointers(xd, fd, ys)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for rep in range(3):
            xs = [rng.integers(-4, 5, size=tuple(x.shape)).astype(np.float32) for x in xd]
            fs = [rng.integers(-4, 5, size=tuple(f.shape)).astype(np.float32) for f in fd]
            for t, a in zip(xd + fd, xs + fs):
                t.copy_(torch.from_numpy(a))
            plan.launch(use_graph=True)
            side.synchronize()
            for y, x, f in zip(ys, xs, fs):
                np.testing.assert_array_equal(host(y), oracle.forward(x, f).astype(np.float32))
