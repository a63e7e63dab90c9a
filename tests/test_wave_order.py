"""Lanes of one wave that exchange values through LDS without a workgroup
barrier need an order that the compiler keeps: wave_order(), a release and an
acquire fence of wavefront scope.  A wave barrier alone orders no memory."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0912_0180_amd", "csrc")
KERNELS = open(os.path.join(CSRC, "hh_kernels.hpp")).read()
IDR = open(os.path.join(CSRC, "hh_idr_kernels.hpp")).read()


def body(src, start):
    src = src[src.index(start):]
    return src[: src.index("\n}\n")]


def test_wave_order_is_a_pair_of_fences():
    b = body(KERNELS, "void wave_order()")
    assert re.search(r"fence\(__ATOMIC_RELEASE, \"wavefront\"\);.*fence\(__ATOMIC_ACQUIRE, \"wavefront\"\);", b, re.S)
    # no other place relies on the bare barrier
    assert (KERNELS + IDR).count("__builtin_amdgcn_wave_barrier") == 1


def test_row_form_orders_its_ring():
    """The solving wave writes a step's values and reads them one step later."""
    b = body(KERNELS, "void ilu_stage(")
    assert len(re.findall(r"\n *cur\[s \* ST [^;]*;", b)) == 1
    assert re.search(r"\n *cur\[s \* ST [^;]*;\s*wave_order\(\);", b)


def test_idr_finaliser_orders_its_small_solve():
    b = body(IDR, "void idr_finalize(")
    assert re.search(r"wave_order\(\);[^;]*\n\s*if \(!small_solve", b)
    assert re.search(r"step\(\);\s*wave_order\(\);[^;]*\n\s*if \(t == 0\) \{", b)
