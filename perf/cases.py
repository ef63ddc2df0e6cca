"""Timed cases of the framework: the calls that its users make, over the range
of sizes, element types and options that they make them with.

A case is a dict of plain values:

* ``kind`` "forward": one filter-bank correlation, y = plan.forward(x, w);
  ``epilogue`` is an elementwise expression fused into its store (or "").
* ``kind`` "step": forward and both gradients through autograd, as a training
  step calls them.
* ``kind`` "batched": many uneven images, each with its own bank, in one
  launch; the shapes are drawn from ``shape_seed``.
* ``kind`` "nearest": exact nearest neighbours of 8-bit patches.

Inputs are made on the GPU from the seed alone: images uniform in [-1, 1],
filters with zero mean and unit norm, upstream gradients standard normal,
patches cut from images with a 1/f amplitude spectrum.
"""
import math
import random

import torch

from paper_0911_3456_amd import BatchedPlan, NNPlan, Plan, fbcorr
from paper_0911_3456_amd.plan import get_plan

CLAMP = "fminf(fmaxf(v, 0.f), 1.f)"


def _corr(name, kind, batch, H, W, D, N, fh, fw, precision="fp32", epilogue=""):
    return {"name": name, "kind": kind, "batch": batch, "H": H, "W": W, "D": D, "N": N, "fh": fh, "fw": fw,
            "precision": precision, "epilogue": epilogue}


def listed():
    return [
        # the smallest call: one small image, a small bank (launches and host time)
        _corr("tiny_forward", "forward", 1, 64, 64, 4, 16, 5, 5),
        # a first layer on one colour picture, with the clamp that follows it
        _corr("colour_clamped", "forward", 1, 480, 640, 3, 32, 7, 7, epilogue=CLAMP),
        # a large picture with a narrow bank (from the paper's tuning table)
        _corr("large_narrow", "forward", 1, 1024, 1024, 8, 16, 5, 5),
        # one image of the paper's table, trained
        _corr("table_step", "step", 1, 256, 256, 8, 64, 9, 9),
        # the benchmark's training step: a batch that fills the chip
        _corr("train_step", "step", 32, 128, 128, 16, 64, 7, 7),
        # a training step at sizes that are multiples of nothing
        _corr("ragged_step", "step", 6, 97, 131, 24, 48, 5, 3),
        # the 16-bit forward of a wide bank of large filters
        _corr("wide_bf16", "forward", 1, 512, 512, 16, 128, 13, 13, precision="bf16"),
        # a ragged batch in the other 16-bit type, small filters
        _corr("ragged_fp16", "forward", 3, 201, 157, 32, 96, 5, 5, precision="fp16"),
        # uneven images with their own banks, one launch
        {"name": "uneven_batch", "kind": "batched", "count": 32, "shape_seed": 1},
        # entropy estimation: the search at both ends of its range of sizes ...
        {"name": "nearest_small", "kind": "nearest", "T": 4096, "M": 4096, "side": 8},
        {"name": "nearest_large", "kind": "nearest", "T": 4096, "M": 1048576, "side": 8},
        # ... and with other patches and sizes that are multiples of nothing
        {"name": "nearest_ragged", "kind": "nearest", "T": 1003, "M": 77777, "side": 12},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# The largest correlation drawn: products of one pass, and elements of one tensor.
MAX_FLOPS = 1.2e11
MAX_ELEMS = 3.0e7


def draw(rng):
    kind = rng.choice(["forward", "forward", "step", "step", "lowp", "batched", "nearest"])
    if kind == "batched":
        return {"kind": "batched", "count": _log(rng, 4, 20), "shape_seed": rng.randrange(1 << 20)}
    if kind == "nearest":
        while True:
            T, M, side = _log(rng, 64, 8192), _log(rng, 1024, 1 << 20), rng.choice([4, 8, 8, 12, 16])
            if T * M * side * side <= 4096 * 1048576 * 64:
                return {"kind": "nearest", "T": T, "M": M, "side": side}
    while True:
        batch = rng.choice([1, 1, _log(rng, 1, 32)])
        H, W = _log(rng, 48, 1024), _log(rng, 48, 1024)
        D = rng.choice([1, 3, 4, 8, 16, 32, _log(rng, 1, 64)])
        N = rng.choice([16, 32, 64, 128, _log(rng, 4, 160)])
        fh = rng.choice([3, 5, 7, 9, 11, 13, rng.randint(1, 13)])
        fw = rng.choice([fh, fh, rng.randint(1, 13)])
        case = _corr("", "step" if kind == "step" else "forward", batch, H, W, D, N, fh, fw,
                     precision=rng.choice(["bf16", "fp16"]) if kind == "lowp" else "fp32",
                     epilogue=CLAMP if kind != "step" and rng.random() < 0.25 else "")
        out = batch * (H - fh + 1) * (W - fw + 1) * N
        if work(case)["flops"] <= MAX_FLOPS and max(batch * H * W * D, out) <= MAX_ELEMS:
            del case["name"]
            return case


def _batch_shapes(case):
    """(H, W, D, N, fh, fw) of every image."""
    rng = random.Random(case["shape_seed"])
    out = []
    for _ in range(case["count"]):
        f = rng.choice([3, 5, 7, 9, 11])
        out.append((rng.randint(96, 512), rng.randint(96, 512), rng.choice([3, 4, 8, 16, 32]),
                    rng.choice([16, 32, 64, 128]), f, f))
    return out


def _corr_shapes(case):
    B, H, W, D, N, fh, fw = (case[k] for k in ("batch", "H", "W", "D", "N", "fh", "fw"))
    return (B, H, W, D), (N, fh, fw, D), (B, H - fh + 1, W - fw + 1, N)


def work(case):
    if case["kind"] == "nearest":
        T, M, dim = case["T"], case["M"], case["side"] ** 2
        return {"bytes": (T + M) * dim + 8 * T, "flops": 2 * T * M * dim}
    if case["kind"] == "batched":
        nbytes = flops = 0
        for H, W, D, N, fh, fw in _batch_shapes(case):
            out = (H - fh + 1) * (W - fw + 1) * N
            nbytes += 4 * (H * W * D + N * fh * fw * D + out)
            flops += 2 * out * fh * fw * D
        return {"bytes": nbytes, "flops": flops}
    xs, ws, ys = _corr_shapes(case)
    flops = 2 * math.prod(ys) * math.prod(ws[1:])
    nbytes = 4 * (math.prod(xs) + math.prod(ws) + math.prod(ys))
    # a step reads x, w and dy and writes y, dx and dw
    return {"bytes": 2 * nbytes, "flops": 3 * flops} if case["kind"] == "step" else {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _image(gen, shape):
    return torch.rand(shape, device="cuda", generator=gen).mul_(2).sub_(1)


def _bank(gen, shape):
    w = torch.rand(shape, device="cuda", generator=gen, dtype=torch.float64).mul_(2).sub_(1)
    flat = w.view(shape[0], -1)
    if flat.shape[1] > 1:
        flat = flat - flat.mean(dim=1, keepdim=True)
    flat = flat / flat.norm(dim=1, keepdim=True).clamp_min(1e-30)
    return flat.view(shape).float()


def _patches(gen, count, side):
    """count patches [count, side*side] of 8-bit pixels."""
    size, per_image = 512, 16384
    freq = torch.fft.fftfreq(size, device="cuda")[:, None].hypot(torch.fft.rfftfreq(size, device="cuda")[None, :])
    freq[0, 0] = 1.0
    out = torch.empty((count, side, side), dtype=torch.uint8, device="cuda")
    off = torch.arange(side, device="cuda")
    for lo in range(0, count, per_image):
        n = min(per_image, count - lo)
        spec = torch.fft.rfft2(torch.randn((size, size), device="cuda", generator=gen)) / freq
        spec[0, 0] = 0
        img = torch.fft.irfft2(spec, s=(size, size))
        img = (128 + 48 * (img - img.mean()) / img.std()).round().clamp(0, 255).to(torch.uint8)
        pos = torch.randint(0, size - side + 1, (2, n), device="cuda", generator=gen)
        out[lo:lo + n] = img[pos[0][:, None, None] + off[:, None], pos[1][:, None, None] + off]
    return out.view(count, side * side)


def _inputs(case, seed):
    gen = _generator(seed)
    if case["kind"] == "nearest":
        return _patches(gen, case["T"], case["side"]), _patches(gen, case["M"], case["side"])
    if case["kind"] == "batched":
        shapes = _batch_shapes(case)
        return ([_image(gen, (H, W, D)) for H, W, D, N, fh, fw in shapes],
                [_bank(gen, (N, fh, fw, D)) for H, W, D, N, fh, fw in shapes])
    xs, ws, ys = _corr_shapes(case)
    x, w = _image(gen, xs), _bank(gen, ws)
    if case["kind"] == "step":
        return x, w, torch.randn(ys, device="cuda", generator=gen)
    return x, w


def prepare(case, seed):
    """Inputs, and the plan that a program keeps."""
    state = {"kind": case["kind"], "inputs": _inputs(case, seed)}
    if case["kind"] == "nearest":
        state["plan"] = NNPlan(case["T"], case["M"], case["side"] ** 2)
        return state
    if case["kind"] == "batched":
        state["plan"] = BatchedPlan(_batch_shapes(case))
        state["out"] = state["plan"].output_buffers()
        return state
    shape = [case[k] for k in ("batch", "H", "W", "D", "N", "fh", "fw")]
    if case["kind"] == "step":
        x, w, _ = state["inputs"]
        x.requires_grad_(True)
        w.requires_grad_(True)
        plan = get_plan(*shape)
        plan.workspace_size(1)            # the gradients' kernels, compiled once
        return state
    state["plan"] = Plan(*shape, precision=case["precision"])
    if case["epilogue"]:
        state["plan"].set_epilogue(case["epilogue"])
    return state


def run(state):
    if state["kind"] == "nearest":
        return state["plan"].search(*state["inputs"])
    if state["kind"] == "batched":
        xs, ws = state["inputs"]
        return state["plan"].forward(xs, ws, state["out"])
    if state["kind"] == "step":
        x, w, dy = state["inputs"]
        y = fbcorr(x, w)
        dx, dw = torch.autograd.grad(y, (x, w), dy)
        return y.detach(), dx, dw
    x, w = state["inputs"]
    return state["plan"].forward(x, w)


# ---------------------------------------------------------------- 64 bits

def _windows(x, u, ho, wo, fw):
    """[rows, fw*D]: for filter row u, the window of every output pixel."""
    B, H, W, D = x.shape
    v = x[:, u:u + ho].as_strided((B, ho, wo, fw * D), (H * W * D, W * D, D, 1), x.storage_offset() + u * W * D)
    return v.reshape(B * ho * wo, fw * D)


def _slabs(x, ho, fh, wo, k):
    """Output row ranges whose windows stay below about a gigabyte."""
    step = max(1, int(1.2e8 // (x.shape[0] * wo * k)))
    return [(i, min(i + step, ho)) for i in range(0, ho, step)]


def _exact_corr(x, w):
    x, w = x.double().contiguous(), w.double()
    N, fh, fw, D = w.shape
    B, ho, wo = x.shape[0], x.shape[1] - fh + 1, x.shape[2] - fw + 1
    y = torch.zeros((B, ho, wo, N), dtype=torch.float64, device=x.device)
    for i, j in _slabs(x, ho, fh, wo, fw * D):
        part = x[:, i:j + fh - 1].contiguous()
        acc = torch.zeros((B * (j - i) * wo, N), dtype=torch.float64, device=x.device)
        for u in range(fh):
            acc.addmm_(_windows(part, u, j - i, wo, fw), w[:, u].reshape(N, fw * D).t())
        y[:, i:j] = acc.view(B, j - i, wo, N)
    return y


def _exact_dx(w, dy):
    N, fh, fw, D = w.shape
    padded = torch.nn.functional.pad(dy, (0, 0, fw - 1, fw - 1, fh - 1, fh - 1))
    return _exact_corr(padded, w.flip(1, 2).permute(3, 1, 2, 0).contiguous())


def _exact_dw(x, dy, fh, fw):
    x, dy = x.double().contiguous(), dy.double()
    B, ho, wo, N = dy.shape
    D = x.shape[3]
    dw = torch.zeros((N, fh, fw, D), dtype=torch.float64, device=x.device)
    for i, j in _slabs(x, ho, fh, wo, fw * D):
        part, g = x[:, i:j + fh - 1].contiguous(), dy[:, i:j].reshape(-1, N).t()
        for u in range(fh):
            dw[:, u] += (g @ _windows(part, u, j - i, wo, fw)).view(N, fw, D)
    return dw


def _exact_nearest(targets, neighbours):
    t, step = targets.double(), 32768
    best = torch.full((t.shape[0],), float("inf"), dtype=torch.float64, device=t.device)
    tt = (t * t).sum(dim=1, keepdim=True)
    for lo in range(0, neighbours.shape[0], step):
        n = neighbours[lo:lo + step].double()
        d = tt + (n * n).sum(dim=1) - 2 * (t @ n.t())
        # distance, then index: both below 2^53 together
        key = d * 2.0 ** 21 + torch.arange(lo, lo + n.shape[0], dtype=torch.float64, device=t.device)
        best = torch.minimum(best, key.amin(dim=1))
    dist = (best / 2.0 ** 21).floor()
    return (best - dist * 2.0 ** 21).to(torch.int32), dist.to(torch.int32)


def exact(case, seed):
    inputs = _inputs(case, seed)
    if case["kind"] == "nearest":
        return _exact_nearest(*inputs)
    if case["kind"] == "batched":
        return [_exact_corr(x[None], w)[0] for x, w in zip(*inputs)]
    x, w = inputs[:2]
    y = _exact_corr(x, w)
    if case["kind"] == "step":
        return y, _exact_dx(w, inputs[2]), _exact_dw(x, inputs[2], case["fh"], case["fw"])
    return y.clamp(0, 1) if case["epilogue"] else y
