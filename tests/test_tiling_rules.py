"""The tiling rules' choices build: for every problem of a random sample, a
role that the rule gives to the three-part or 16-bit register-streamed kernels
gets them (a choice that the generator refuses would silently fall back)."""
import numpy as np
import pytest

from paper_0911_3456_amd import FbcorrError, codegen, make_desc


def _sample(seed, n):
    rng = np.random.default_rng(seed)
    for _ in range(n):
        fh, fw = (int(v) for v in rng.integers(1, 14, 2))
        H, W = fh + int(2 ** rng.uniform(0, 9)) - 1, fw + int(2 ** rng.uniform(0, 9)) - 1
        yield (int(rng.integers(1, 9)), H, W, int(2 ** rng.uniform(0, 7)), int(2 ** rng.uniform(0, 8)), fh, fw)


def _staged_slices(role, lowp, cin, cout, win):
    if role == "backward_x":
        return cout > 16 and (win == 1 or (cin <= 8 and win <= 5))
    if not lowp:
        return win == 1 or win * cin < 36
    return (cout % 4 != 0 and 0.5 * win * cin * cout / (cin + cout) < 12) or (win == 1 and cin % 4 != 0 and cin > 16)


def test_correlations():
    seen = set()
    for s in _sample(21, 200):
        B, H, W, D, N, fh, fw = s
        win, flops = fh * fw, 2.0 * B * (H - fh + 1) * (W - fw + 1) * N * fh * fw * D
        for prec in ("bf16", "fp16"):
            want = not _staged_slices("forward", True, D, N, win)
            assert ("rgemm" in codegen(make_desc(*s, precision=prec), "forward", None)[1]) == want, (s, prec)
            seen.add((prec, want))
        want = not _staged_slices("backward_x", False, N, D, win)
        assert ("-DFB_DT=3" in codegen(make_desc(*s), "backward_x", None)[1]) == want, s
        seen.add(("dx", want))
        parts = flops >= 2e8 and win * D > (64 if D == 1 else 16) and not _staged_slices("forward", False, D, N, win)
        _, o = codegen(make_desc(*s), "forward", None)
        if parts and "-DFB_DT=3" not in o:
            # only a bank past the static scratch (16 MiB) stays on fp32 instructions
            assert N * win * D * 6 > 8 << 20, s
        else:
            assert ("-DFB_DT=3" in o) == parts, s
        seen.add(("fp32", parts))
    assert {("bf16", True), ("bf16", False), ("dx", True), ("dx", False), ("fp32", True), ("fp32", False)} <= seen


def test_filter_gradients():
    """dws wherever dw accepts the size and some tiling fits (rows of many odd
    channels are staged in four copies: then none may)."""
    n, none = 0, 0
    for s in _sample(22, 200):
        d = make_desc(*s)
        try:
            codegen(d, "backward_w", "algo=dw")
        except FbcorrError:
            continue
        if "-DFB_RSEG" in codegen(d, "backward_w", None)[1]:
            n += 1
            continue
        with pytest.raises(FbcorrError, match="every knob"):
            codegen(d, "backward_w", "algo=dws")
        assert s[3] % 4 and s[3] > 36, s
        none += 1
    assert n > 150 and none > 0
