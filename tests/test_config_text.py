"""Configuration texts that leave knobs out (host only): an algorithm's name
alone is a complete configuration for every role it serves, and a text without
an algorithm starts from the database's entry for the problem, also where that
entry is kept beside another default."""
import re

import pytest

STEP = (32, 128, 128, 16, 64, 7, 7)       # entries for rgemm (forward, dX) and dw


def _opts(shape, role, cfg, **kw):
    from paper_0911_3456_amd import codegen, make_desc
    return {k: int(v) for k, v in re.findall(r"-DFB_(\w+)=(-?\d+)", codegen(make_desc(*shape, **kw), role, cfg)[1])}


@pytest.mark.parametrize("shape", [STEP, (1, 40, 50, 3, 20, 5, 4), (2, 33, 41, 24, 100, 3, 3), (1, 9, 11, 5, 33, 9, 11)])
def test_dws_alone(shape):
    o = _opts(shape, "backward_w", "algo=dws")
    assert o["RSEG"] >= 1 and o["RT"] >= 1
    assert _opts(shape, "backward_w", "algo=dws np=1")["NP"] == 1
    one = _opts(shape, "backward_w", "algo=dws rt=1")
    assert one["RT"] == 1 and one["RW"] == o["RW"]


@pytest.mark.parametrize("role,names", [("forward", ("igemm", "rgemm", "direct")), ("backward_x", ("igemm", "rgemm")),
                                        ("backward_w", ("dw", "dws"))])
def test_every_name_alone(role, names):
    for shape in (STEP, (1, 40, 50, 3, 20, 5, 4), (1, 30, 30, 32, 48, 3, 3)):
        for n in names:
            _opts(shape, role, "algo=" + n)


def test_no_algorithm_starts_from_the_entry():
    o = _opts(STEP, "forward", "pf=1")
    assert o["PF"] == 1 and (o["NT"], o["MT"], o["WPE"], o["STE"]) == (4, 4, 1, 1)
    o = _opts(STEP, "backward_x", "pf=2")
    assert o["PF"] == 2 and (o["MT"], o["WM"]) == (8, 4)
    o = _opts((1, 256, 256, 8, 64, 9, 9), "backward_w", "np=100")
    assert o["NP"] == 100 and (o["RW"], o["TPB"]) == (62, 21)
    o = _opts((1, 256, 256, 8, 64, 9, 9), "forward", "wpad=4")
    assert o["WPAD"] == 4 and (o["MT"], o["USTAGE"]) == (2, 3)
    # without an entry: the kernels that fit any size, as ever
    assert _opts((1, 100, 100, 16, 64, 7, 7), "forward", "wpad=8")["WPAD"] == 8
    assert _opts((1, 100, 100, 16, 64, 7, 7), "backward_w", "np=3")["NP"] == 3
