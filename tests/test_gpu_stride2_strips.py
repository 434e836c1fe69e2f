"""The stride-2 strips of four outputs a lane (conv2d_fbs_stride2_strip_kernel): single rows of every width, and images of one to three columns, into a pitched output
whose surroundings stay untouched, from a region of a wider image of NaN.  test_stride2_rules.py checks without a GPU that these images reach all kernels."""
import pytest

from test_gpu_stride2_pairs import run_in_a_region

pytestmark = pytest.mark.gpu

SINGLE_ROW_IMAGES = [(701, 515), (64, 1031), (1, 16)]                      # a whole strip (at most 512 input columns) and a cut one, two and a cut one, the smallest
NARROW = [(w, kh, kw) for w, kw in ((1, 1), (2, 1), (3, 1), (2, 2), (3, 2), (3, 3)) for kh in (2, 9, 15)]
NARROW_ROWS = [5, 4097, 4098, 100001, 100002, 100003]                      # one, two and three rows a wavefront, with and without some left over


@pytest.mark.parametrize("kw", range(1, 16))
@pytest.mark.parametrize("h,w", SINGLE_ROW_IMAGES)
def test_single_rows_of_every_width(h, w, kw):
    run_in_a_region(1, kw, h, w)


@pytest.mark.parametrize("w,kh,kw", NARROW)
@pytest.mark.parametrize("oh", NARROW_ROWS)
def test_narrow_images(oh, w, kh, kw):
    run_in_a_region(kh, kw, 2 * (oh - 1) + kh + oh % 2, w)
