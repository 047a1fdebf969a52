"""A caller's block keeps its use: the workspace of a context (lc_workspace_query) does not outgrow the sizes that
earlier versions of the library asked for, which a program may have fixed.  Host only."""
import ctypes as C

import pytest

# grid, and the bytes for basis length 40 before the transforms had packed factors of their own
SIZES = [((2, 2, 2), 397824), ((16, 14, 12), 6995200), ((16, 16, 16), 10266368), ((64, 64, 64), 592895744),
         ((97, 121, 65), 1715192320), ((100, 100, 100), 2243071744), ((128, 128, 128), 4689470720),
         ((200, 200, 200), 17819244288), ((256, 256, 256), 37311791360), ((257, 40, 30), 717235712),
         ((1024, 16, 16), 907719168), ((300, 300, 300), 59999731200)]


@pytest.mark.parametrize("dims,before", SIZES)
def test_workspace_fits_an_earlier_block(dims, before):
    from paper_1704_08521_amd import _lib as L
    b = C.c_size_t()
    assert L.load().lc_workspace_query(*dims, 40, C.byref(b)) == L.LC_OK
    assert 0.7 * before < b.value <= before
