"""Launch grids: only the x side may grow with the problem set (2^31 - 1
workgroups); the y side takes 65,535, and a batch may have more problems."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0912_0180_amd", "csrc")


def test_y_side_holds_values_not_problems():
    sides = []
    for f in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        for m in re.finditer(r"dim3\(([^,()]*(?:\([^()]*\)[^,()]*)*),([^()]*(?:\([^()]*\)[^()]*)*)\)", open(f).read()):
            sides.append((os.path.basename(f), m.group(1).strip(), m.group(2).strip()))
    assert sides                           # the finaliser's sums by value
    for name, x, y in sides:
        words = set(re.findall(r"[A-Za-z_]\w*", y))
        assert words <= {"step", "HH_MAX_S", "ns", "nv"}, (name, x, y)   # s and values per problem, at most 33
