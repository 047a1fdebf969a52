"""Stencil and fused correction where a block marches over several planes, and the stencil's rows of 8 and 16 lanes.

Small grids take chunks of one plane.  These sizes take more, most of them with a shorter last chunk (lanes per row:
planes per chunk, planes of the last one):

* stencil, 8 lanes (3, 256, 256) 5, 2; (28, 203, 150) 7, 4; (35, 180, 99) 4, 4; 16 lanes (12, 200, 203) 6, 6;
  (27, 250, 103) 4, 4; (61, 150, 150) 9, 7; (13, 421, 216) 13, 9; 32 lanes (97, 121, 65) 5, 1; (59, 250, 90) 6, 1;
  (100, 100, 100) 6, 5; (119, 301, 61) 11, 7; (40, 516, 77) 12, 6;
* correction (3, 256, 256) 8, 8; (11, 256, 200) 7, 4; (12, 200, 203) 6, 5; (28, 203, 150) 4, 2; (97, 121, 65) 3, 2;
  (100, 100, 100) 3, 1.

Rows of 8 lanes hold 12 faces and blocks 32 rows, of 16 lanes 28 faces and 16 rows: sizes on both sides of one and
of several tiles.  Checks and tolerances are those of the tests of the tile edges.
"""
import pytest

from tests.test_gpu_correction_tiles import test_pass_against_separate_calls as check_correction
from tests.test_gpu_stencil_tiles import test_momentum_tile_edges as check_stencil

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(3, 256, 256), (28, 203, 150), (35, 180, 99), (12, 200, 203), (27, 250, 103),
                                  (61, 150, 150), (13, 421, 216), (97, 121, 65), (59, 250, 90), (100, 100, 100),
                                  (119, 301, 61), (40, 516, 77)])
def test_stencil_marches(dims):
    check_stencil(dims)


@pytest.mark.parametrize("dims", [(10, 31, 3), (11, 32, 2), (12, 15, 4), (23, 33, 3), (24, 16, 5), (26, 17, 2), (27, 15, 3),
                                  (28, 31, 2), (34, 32, 3), (35, 63, 2), (36, 7, 3), (55, 9, 2), (83, 47, 2), (84, 16, 3)])
def test_stencil_short_rows(dims):
    check_stencil(dims)


@pytest.mark.parametrize("dims", [(3, 256, 256), (11, 256, 200), (12, 200, 203), (28, 203, 150), (97, 121, 65),
                                  (100, 100, 100)])
def test_correction_marches(dims):
    check_correction(dims)
