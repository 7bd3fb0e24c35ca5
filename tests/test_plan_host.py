"""Plans of the nested dissection (host only): every launch fits a compute unit.

A level of narrow fronts asks for LDS that grows with its widest front.  The
boxes of about 60 to 65 nodes a side halve into the widest ones (29 to 32
pivots, a ring of 177 to 192): squares of 241 to 260, 481 to 520 and 961 to
1040 nodes a side have them, and rectangles near those.
"""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2301_10762_amd", "libhelm.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libhelm.so not built")

LDS = 160 * 1024


def _lds(nx, nz):
    from paper_2301_10762_amd import helm
    out = (ctypes.c_size_t * 4)()
    assert helm.lib().helm_plan_lds(ctypes.byref(helm._Grid(nx, nz, 1.0, 1.0)), out) == 0
    return list(out)


def test_squares_fit_lds():
    for n in [*range(2, 521), 961, 1000, 1024, 1040]:
        assert max(_lds(n, n)) <= LDS, (n, _lds(n, n))


@pytest.mark.parametrize("part", range(4))
def test_rectangles_fit_lds(part):
    for nx in range(33 + 7 * part, 402, 28):
        for nz in [*range(35, 402, 11), 2 * nx, 2 * nx - 5, 3 * nx]:
            assert max(_lds(nx, nz)) <= LDS, (nx, nz, _lds(nx, nz))
