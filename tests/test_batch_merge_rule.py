"""Where a 2D batch takes the merged legs (batch_merge_pays, compiled for the
host): the sides of the line that measuring both routes gave, batch by batch."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "hh_merge.h"
extern "C" int pays(const hh::BatchShape *p, int n, int fp32) { return hh::batch_merge_pays(p, n, fp32 != 0); }
"""


class Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("on", "levels", "tail", "split", "kdown", "kup")] + [
        ("down", ctypes.c_long), ("up", ctypes.c_long)]


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(SRC)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I",
                        os.path.join(ROOT, "paper_0912_0180_amd", "csrc"), str(d / "rule.cpp"), "-o", str(d / "rule.so")],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(str(d / "rule.so")).pays


def ceil(a, b):
    return -(-a // b)


def shape(n, levels, fp32):
    side = [[v >> l for v in n] for l in range(levels)]
    size = [a * b for a, b in side]
    s = Shape()
    s.levels = levels
    s.tail = next((l for l in range(1, levels) if size[l] <= 1024), levels - 1)   # of the sizes here, all fit its LDS
    s.split = size[-1] > 128
    s.kdown, s.kup = min(3, levels - 2), min(4, levels - 2)
    s.on = s.kdown >= 2
    C, UT = (3 if fp32 else 2), (32 if s.kup == 4 else 16)
    s.down = ceil(side[-1][0], C) * ceil(side[-1][1], C)
    u = side[levels - 1 - s.kup]
    s.up = ceil(u[0], UT) * ceil(u[1], UT)
    return s


# problems (sides, levels), and whether the merged legs were faster in FP64, FP32
MEASURED = [
    ([((416, 416), 5)] * 2, False, True),                             # 338 FP64 workgroups, no tail kernel saved
    ([((368, 336), 5)] * 2, False, True),
    ([((352, 352), 5)] * 3, False, True),
    ([((320, 320), 5)] * 4, False, True),
    ([((640, 400), 5)] * 2, False, True),                             # 520
    ([((432, 432), 5)] * 3, False, True),                             # 588
    ([((272, 272), 5)] * 7, False, None),
    ([((240, 272), 5)] * 8, False, None),                             # 576, tail kernels saved
    ([((864, 864), 6)] * 3, False, None),
    ([((352, 320), 5)] * 2, True, None),                              # one round
    ([((288, 288), 5)] * 3, True, None),
    ([((192, 192), 5)] * 2, True, True),
    ([((192, 192), 5)] * 10, True, True),                             # two rounds, tail kernels saved
    ([((256, 256), 5)] * 6, True, True),
    ([((512, 512), 6)] * 7, True, True),
    ([((864, 864), 6)] * 2, True, True),                              # two rounds, five launches saved
    ([((1728, 1728), 7)] * 2, True, True),
    ([((960, 960), 6), ((480, 480), 5)], True, None),
    ([((400, 400), 5)] + [((256, 256), 5)] * 3, True, None),
    ([((480, 480), 5)] + [((128, 128), 4)] * 2, True, None),
    ([((320, 320), 5), ((160, 160), 4)] * 2, True, None),
    ([((512, 512), 5), ((256, 256), 4)], False, None),
    ([((512, 512), 5), ((256, 256), 6)], True, None),                 # a whole tail kernel saved
    ([((512, 512), 5), ((512, 512), 7)], False, True),
    ([((256, 256), 4)] + [((256, 256), 6)] * 3, True, True),
    ([((256, 256), 4)] * 2, True, True),                              # two merged levels
    ([((128, 128), 4)] * 7, True, True),
    ([((128, 128), 4)] * 2 + [((128, 128), 5)], True, True),
    ([((352, 320), 5)] * 2 + [((96, 80), 3)], False, True),           # beside one that keeps its launches
    ([((400, 400), 5)] * 2 + [((96, 80), 3)], False, True),
    ([((400, 400), 5)] * 2 + [((64, 64), 2)], False, True),
    ([((768, 768), 6)] * 2 + [((112, 112), 3)], False, True),
    ([((128, 160), 4), ((96, 80), 3)], False, False),
    ([((144, 144), 4)] * 3 + [((96, 80), 3)], False, False),
    ([((160, 160), 4)] * 2 + [((112, 112), 3)], False, False),
    ([((192, 192), 4)] * 2 + [((64, 64), 3)], True, True),
    ([((256, 256), 5), ((48, 40), 3)], True, True),
    ([((256, 256), 5), ((128, 128), 3)], True, True),
    ([((1024, 1024), 7), ((112, 112), 3)], True, True),
    ([((1024, 1024), 7), ((48, 40), 3)], True, True),
    ([((1024, 1024), 8), ((128, 128), 4)], True, True),
]


@pytest.mark.parametrize("case", range(len(MEASURED)))
def test_rule_takes_the_faster_route(pays, case):
    problems, f64, f32 = MEASURED[case]
    for fp32, want in ((0, f64), (1, f32)):
        if want is not None:
            A = (Shape * len(problems))(*[shape(n, l, fp32) for n, l in problems])
            assert bool(pays(A, len(problems), fp32)) == want, (problems, fp32)
