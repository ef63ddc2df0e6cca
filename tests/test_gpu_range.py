"""Ranges of values inside one tensor: filters that mix a large and a tiny
tap, with the input zero under the large one, so that the outputs are the
tiny products alone.  Every element within the fp32 bound of its own sum of
magnitudes, for the forward pass, the input gradient (whose columns contract
over the filters) and the batched launch."""
import numpy as np
import pytest

from _gpu_util import host, need_gpu, to_dev

pytestmark = pytest.mark.gpu

TOL = 1e-5          # the fp32 bound of the other tests, of sum |x||w|

# large tap, tiny taps' scale, scale of the inputs under the tiny taps
RANGES = [
    (1.0, 1.23e-36, 1.0),
    (1.0, 1e-42, 1e15),              # subnormal taps
    (1e20, 1.23e-18, 0.77),
    (1e20, 1e-22, 1.0),
    (2.0 ** 60, 1.23, 1.23e-29),
    (2.0 ** 23, 1e-5, 1e-26),        # tiny products of a large filter
    (3000.0, 1e-33, 1e8),
    (3000.0, 1e-20, 1e-10),
    (1e-30, 1e-42, 1e10),
    (1.0, 0.5, 1e-29),
]


def _close(got, ref, scl):
    err = np.abs(got.astype(np.float64) - ref)
    # (last bits below the normal range are as far apart as fp32 has them)
    bad = err > TOL * scl + 2.0 ** -148
    assert not bad.any(), (got[bad][:3], ref[bad][:3])


def _corr(x, w):
    """fp64 correlation of x [B,H,W,D] and its sum of magnitudes."""
    N, fh, fw, D = w.shape
    x, w = x.astype(np.float64), w.astype(np.float64)
    ho, wo = x.shape[1] - fh + 1, x.shape[2] - fw + 1
    ref, scl = np.zeros((x.shape[0], ho, wo, N)), np.zeros((x.shape[0], ho, wo, N))
    for u in range(fh):
        for v in range(fw):
            a, b = x[:, u:u + ho, v:v + wo], w[:, u, v].T
            ref += a @ b
            scl += np.abs(a) @ np.abs(b)
    return ref, scl


def _bank(rng, N, fh, fw, D, big, tiny):
    """Tiny taps; channel 0 of the first tap large, and ordinary last filters."""
    w = rng.standard_normal((N, fh, fw, D)).astype(np.float32)
    w[:N - 4] *= np.float32(tiny)
    w[:N - 4, 0, 0, 0] = big
    return w


@pytest.mark.parametrize("cfg", ["mf=32 kc=8 mr=2 mt=1 nt=1 wm=2 wn=1 pf=2",
                                 "mf=16 kc=8 mr=1 mt=2 nt=2 wm=2 wn=1 pf=2 ste=1"])
@pytest.mark.parametrize("big,tiny,xs", RANGES)
def test_forward(big, tiny, xs, cfg):
    need_gpu()
    from paper_0911_3456_amd import Plan
    rng = np.random.default_rng(5)
    w = _bank(rng, 40, 5, 3, 16, big, tiny)
    x = rng.standard_normal((1, 30, 37, 16)).astype(np.float32) * np.float32(xs)
    x[..., 0] = 0.0
    p = Plan(1, 30, 37, 16, 40, 5, 3)
    p.set_config("forward", "algo=rgemm sp=1 " + cfg)
    _close(host(p.forward(*to_dev(x, w))), *_corr(x, w))


@pytest.mark.parametrize("big,tiny,xs", RANGES)
def test_input_gradient(big, tiny, xs):
    need_gpu()
    from paper_0911_3456_amd import Plan
    rng = np.random.default_rng(6)
    N, fh, fw, D = 24, 5, 3, 16
    w = rng.standard_normal((N, fh, fw, D)).astype(np.float32) * np.float32(tiny)
    w[0, 0, 0] = big                     # every column's filter 0
    g = rng.standard_normal((1, 26, 35, N)).astype(np.float32) * np.float32(xs)
    g[..., 0] = 0.0
    p = Plan(1, 30, 37, D, N, fh, fw)
    assert "sp=1" in p.get_config("backward_x")
    x = np.zeros((1, 30, 37, D), np.float32)
    dx, _ = p.backward(*to_dev(x, w, g), need_dw=False)
    ref, scl = _corr(np.pad(g, ((0, 0), (fh - 1, fh - 1), (fw - 1, fw - 1), (0, 0))),
                     np.ascontiguousarray(w[:, ::-1, ::-1].transpose(3, 1, 2, 0)))
    _close(host(dx), ref, scl)


@pytest.mark.parametrize("big,tiny,xs", RANGES)
def test_batched(big, tiny, xs):
    need_gpu()
    from paper_0911_3456_amd import BatchedPlan
    rng = np.random.default_rng(7)
    shapes = [(30, 37, 16, 40, 5, 3), (21, 50, 16, 40, 5, 3)]
    xs_, ws = [], []
    for H, W, D, N, fh, fw in shapes:
        x = rng.standard_normal((H, W, D)).astype(np.float32) * np.float32(xs)
        x[..., 0] = 0.0
        xs_.append(x)
        ws.append(_bank(rng, N, fh, fw, D, big, tiny))
    plan = BatchedPlan(shapes)
    assert "sp=1" in plan.describe()
    for x, w, y in zip(xs_, ws, plan.forward(list(to_dev(*xs_)), list(to_dev(*ws)))):
        _close(host(y)[None], *_corr(x[None], w))


# ------------------------------------------------------------ small tails

def _tails(rng, shape, density=0.004):
    """Ordinary values with a few tiny ones, down to the subnormal range."""
    a = rng.standard_normal(shape).astype(np.float32)
    m = rng.random(shape) < density
    a[m] *= (2.0 ** rng.uniform(-148, -100, size=int(m.sum()))).astype(np.float32)
    return a


def _times(fns, reps=10, rounds=5):
    """Best time of each call, taken in turn."""
    import torch
    best = [1e9] * len(fns)
    for f in fns:
        f()
    for _ in range(rounds):
        for k, f in enumerate(fns):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(reps):
                f()
            b.record()
            torch.cuda.synchronize()
            best[k] = min(best[k], a.elapsed_time(b) / reps)
    return best


def test_tails_forward_and_input_gradient():
    """The values' own accuracy, at the rate of ordinary values."""
    need_gpu()
    from paper_0911_3456_amd import Plan
    rng = np.random.default_rng(8)
    B, H, W, D, N, fh, fw = 4, 64, 66, 16, 64, 7, 7
    p = Plan(B, H, W, D, N, fh, fw)
    assert "sp=1" in p.get_config("forward") and "sp=1" in p.get_config("backward_x")
    w = (rng.standard_normal((N, fh, fw, D)) * 0.03).astype(np.float32)
    x, g = _tails(rng, (B, H, W, D)), _tails(rng, (B, H - fh + 1, W - fw + 1, N))
    x[1], g[1] = x[1] * np.float32(1e-38), g[1] * np.float32(1e-38)      # an image of subnormal numbers
    xt, wt, gt = to_dev(x, w, g)
    _close(host(p.forward(xt, wt)), *_corr(x, w))
    dx, _ = p.backward(xt, wt, gt, need_dw=False)
    _close(host(dx), *_corr(np.pad(g, ((0, 0), (fh - 1, fh - 1), (fw - 1, fw - 1), (0, 0))),
                            np.ascontiguousarray(w[:, ::-1, ::-1].transpose(3, 1, 2, 0))))
    x0, g0 = to_dev(rng.standard_normal(x.shape).astype(np.float32), rng.standard_normal(g.shape).astype(np.float32))
    a, b = _times([lambda: p.forward(xt, wt), lambda: p.forward(x0, wt)])
    c, d = _times([lambda: p.backward(xt, wt, gt, need_dw=False), lambda: p.backward(x0, wt, g0, need_dw=False)])
    print("forward %.4f and %.4f ms, input gradient %.4f and %.4f ms" % (a, b, c, d))
    assert a < 1.5 * b and c < 1.5 * d


def test_tails_batched():
    need_gpu()
    from paper_0911_3456_amd import BatchedPlan
    rng = np.random.default_rng(9)
    shapes = [(96, 120, 16, 64, 7, 7)] * 8
    plan = BatchedPlan(shapes)
    xs = [_tails(rng, s[:3]) for s in shapes]
    ws = [rng.standard_normal((64, 7, 7, 16)).astype(np.float32) for _ in shapes]
    xt, wt = list(to_dev(*xs)), list(to_dev(*ws))
    _close(host(plan.forward(xt, wt)[3])[None], *_corr(xs[3][None], ws[3]))
    x0 = list(to_dev(*[rng.standard_normal(s[:3]).astype(np.float32) for s in shapes]))
    ys = plan.output_buffers()
    a, b = _times([lambda: plan.forward(xt, wt, ys), lambda: plan.forward(x0, wt, ys)])
    print("%.4f and %.4f ms" % (a, b))
    assert a < 1.5 * b


@pytest.mark.parametrize("shape", [(1, 96, 110, 16, 64, 7, 7), (1, 96, 150, 3, 64, 7, 7)])
def test_huge_values_cost(shape):
    """What the parts cannot hold (here a huge value in every tile) is right,
    and within a small multiple of the time of fp32 instructions."""
    need_gpu()
    from paper_0911_3456_amd import Plan
    rng = np.random.default_rng(10)
    B, H, W, D, N, fh, fw = shape
    p, q = Plan(*shape), Plan(*shape)
    q.set_config("forward", "algo=igemm")
    w = rng.standard_normal((N, fh, fw, D)).astype(np.float32)
    x = rng.standard_normal((B, H, W, D)).astype(np.float32)
    x[:, ::4, ::8, 0] = 3e38
    xt, wt = to_dev(x, w)
    y, y0 = host(p.forward(xt, wt)), host(q.forward(xt, wt))
    ref, scl = _corr(x, w)
    fin = (scl < 3e38)
    _close(y[fin], ref[fin], scl[fin])
    _close(y0[fin], ref[fin], scl[fin])
    a, b = _times([lambda: p.forward(xt, wt), lambda: q.forward(xt, wt)])
    print("%.4f ms, fp32 instructions %.4f ms" % (a, b))
    assert a < 12 * b


def _dw_ref(x, g, fh, fw):
    x, g = x.astype(np.float64), g.astype(np.float64)
    B, ho, wo, N = g.shape
    g2 = g.reshape(-1, N).T
    ref, scl = (np.zeros((N, fh, fw, x.shape[3])) for _ in range(2))
    for u in range(fh):
        for v in range(fw):
            a = x[:, u:u + ho, v:v + wo].reshape(-1, x.shape[3])
            ref[:, u, v], scl[:, u, v] = g2 @ a, np.abs(g2) @ np.abs(a)
    return ref, scl


def _dw_close(got, x, g, fh, fw):
    ref, scl = _dw_ref(x, g, fh, fw)
    err = np.abs(got.astype(np.float64) - ref)
    # (a sum of that many products, each as far off as fp32 has subnormal ones)
    bad = err > TOL * scl + g.shape[0] * g.shape[1] * g.shape[2] * 2.0 ** -149
    assert not bad.any(), (got[bad][:3], ref[bad][:3])


DW = (2, 60, 70, 8, 64, 7, 7)


def _dw_plan(shape=DW):
    from paper_0911_3456_amd import Plan
    p = Plan(*shape)
    assert "dws" in p.get_config("backward_w")
    return p


@pytest.mark.parametrize("sx,sg", [(1.0, 1.0), (1e-25, 1e-14), (1e-18, 1e-18), (1e-30, 1e8), (1e-42, 1e8), (1e9, 1e-44),
                                   (1e12, 1e12), (1e-39, 1e36)])
def test_filter_gradient_scales(sx, sg):
    """Whole tensors far from one: tiny times tiny, tiny times large."""
    need_gpu()
    rng = np.random.default_rng(11)
    B, H, W, D, N, fh, fw = DW
    x = (rng.standard_normal((B, H, W, D)) * sx).astype(np.float32)
    g = (rng.standard_normal((B, H - fh + 1, W - fw + 1, N)) * sg).astype(np.float32)
    w = np.zeros((N, fh, fw, D), np.float32)
    _dw_close(host(_dw_plan().backward(*to_dev(x, w, g), need_dx=False)[1]), x, g, fh, fw)


@pytest.mark.parametrize("shape", [DW, (1, 50, 61, 3, 33, 5, 4)])
def test_tails_filter_gradient(shape):
    need_gpu()
    rng = np.random.default_rng(12)
    B, H, W, D, N, fh, fw = shape
    p = _dw_plan(shape)
    x, g = _tails(rng, (B, H, W, D)), _tails(rng, (B, H - fh + 1, W - fw + 1, N))
    g[..., 3] *= np.float32(1e-38)               # a filter of subnormal gradients
    x[..., 1] *= np.float32(1e-38)
    w = np.zeros((N, fh, fw, D), np.float32)
    big = rng.standard_normal(x.shape).astype(np.float32)
    big[0, 5, 7, 1], big[B - 1, H - 1, W - 1, 0] = 1e25, -1e22
    xt, wt, gt, bt = to_dev(x, w, g, big)
    _dw_close(host(p.backward(xt, wt, gt, need_dx=False)[1]), x, g, fh, fw)
    _dw_close(host(p.backward(bt, wt, gt, need_dx=False)[1]), big, g, fh, fw)
    x0, g0 = to_dev(rng.standard_normal(x.shape).astype(np.float32), rng.standard_normal(g.shape).astype(np.float32))
    q = _dw_plan(shape)
    q.set_config("backward_w", "algo=dw")
    a, b, c, d = _times([lambda: p.backward(xt, wt, gt, need_dx=False), lambda: p.backward(x0, wt, g0, need_dx=False),
                         lambda: p.backward(bt, wt, g0, need_dx=False), lambda: q.backward(bt, wt, g0, need_dx=False)])
    print("tails %.4f, ordinary %.4f, huge %.4f ms, fp32 instructions %.4f" % (a, b, c, d))
    assert a < 1.5 * b and c < 12 * d


# ------------------------------------------------------------ the limits

@pytest.mark.parametrize("side", [0.999, 1.0, 1.5])
def test_limit_of_the_parts(side):
    """Sums of equal signs right below, at and above the largest magnitude
    that the matrix units take, with the largest filters that they take."""
    need_gpu()
    from paper_0911_3456_amd import Plan
    B, H, W, D, N, fh, fw = 1, 40, 50, 16, 40, 5, 3
    xhi = 70 - int(np.ceil(np.log2(fh * fw * D)))
    rng = np.random.default_rng(13)
    x = (rng.uniform(0.99, 1.0, (B, H, W, D)) * side * 2.0 ** xhi).astype(np.float32)
    p = Plan(B, H, W, D, N, fh, fw)
    p.set_config("forward", "algo=rgemm sp=1 mf=32 kc=8 mr=2 mt=1 nt=1 wm=2 wn=1 pf=2")
    for wmax in (2.0 ** 25 * 0.9999, 2.0 ** 25, 2.0 ** -126, 2.0 ** -149):
        w = np.full((N, fh, fw, D), wmax, np.float32)
        _close(host(p.forward(*to_dev(x, w))), *_corr(x, w))


@pytest.mark.parametrize("side", [0.999, 1.0, 1.5])
def test_limit_of_the_filter_gradient(side):
    need_gpu()
    import re
    from paper_0911_3456_amd import codegen, make_desc
    B, H, W, D, N, fh, fw = DW
    o = {k: int(v) for k, v in re.findall(r"-DFB_(\w+)=(\d+)", codegen(make_desc(*DW), "backward_w", None)[1])}
    ho, wo = H - fh + 1, W - fw + 1
    nseg = B * -(-wo // o["RW"]) * -(-ho // o["RSEG"])
    pixels = -(-nseg // o["NP"]) * o["RSEG"] * o["RW"]
    xhi = (127 - 48 - int(np.ceil(np.log2(pixels)))) // 2
    rng = np.random.default_rng(14)
    x = (rng.uniform(0.99, 1.0, (B, H, W, D)) * side * 2.0 ** xhi).astype(np.float32)
    g = (rng.uniform(0.99, 1.0, (B, ho, wo, N)) * side * 2.0 ** xhi).astype(np.float32)
    w = np.zeros((N, fh, fw, D), np.float32)
    _dw_close(host(_dw_plan().backward(*to_dev(x, w, g), need_dx=False)[1]), x, g, fh, fw)
