"""FP64 transforms of lines whose pieces lie in registers (up to 16 and 32 points with mirror symmetry, 16 without): lengths
on both sides of these limits and of a step of four, on every axis.  Checks and tolerances are those of the
tests of the other tiles."""
import pytest

from tests.test_gpu_full_tiles import test_full_left_transform_tiles as check_full
from tests.test_gpu_line_tiles import test_left_transform_tiles as check_left
from tests.test_gpu_x_lines import test_transforms_along_x as check_x

pytestmark = pytest.mark.gpu

LENGTHS = [6, 10, 12, 13, 15, 16, 17, 24, 25, 31, 32, 33]


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("n", LENGTHS)
def test_short_lines(n, axis):
    check_left(n, axis)
    check_full(n, axis)


@pytest.mark.parametrize("symmetric", [True, False])
@pytest.mark.parametrize("n", LENGTHS)
def test_short_lines_along_x(n, symmetric):
    check_x(n, symmetric)
