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
