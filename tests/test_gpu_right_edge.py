"""Right edge of the image in the 2-D kernels: strips that end inside a lane's four columns, one whole strip before or none, and images of
fewer than four columns.  The image is a region of a wider one that is NaN outside, so a column too many shows.

Tolerance: the parity metric's 1e-5 (fp32 sums of at most 144 terms, see gpu_common).
"""
import numpy as np
import pytest
import torch

from gpu_common import TOL, dev, err2d
from paper_2010_15884_amd import binding as B
from paper_2010_15884_amd import workloads as W

pytestmark = pytest.mark.gpu

# every kernel form: static FBS (square, one row, one column), run-time-sized FBS, BFS and SBM in blocks and in strips
KERNELS = [("FBS", 5, 5), ("FBS", 3, 2), ("FBS", 1, 5), ("FBS", 7, 1), ("FBS", 12, 12), ("BFS", 2, 2), ("BFS", 5, 5), ("BFS", 9, 9), ("SBM", 3, 3),
           ("SBM", 7, 7), ("SBM", 8, 8), ("SBM", 11, 11)]


def _check(proj, kh, kw, h, w):
    x, f = W.random_case(100 * kh + kw + w, (h, w), (kh, kw), x_range=(0.0, 1.0))
    big = torch.full((h, w + 9), float("nan"), dtype=torch.float32, device="cuda")
    big[:, :w] = dev(x)
    ybig = torch.full((h - kh + 3, w - kw + 6), float("nan"), dtype=torch.float32, device="cuda")
    B.sys_conv2d(big[:, :w], f, ybig[1:h - kh + 2, 2:w - kw + 3], projection=proj)
    out = ybig.cpu().numpy()
    assert err2d(np.ascontiguousarray(out[1:h - kh + 2, 2:w - kw + 3]), x, f) <= TOL
    out[1:h - kh + 2, 2:w - kw + 3] = np.nan
    assert np.isnan(out).all()


@pytest.mark.parametrize("proj,kh,kw", KERNELS)
@pytest.mark.parametrize("w", [15, 16, 17, 18, 254, 255, 256, 257, 258, 259, 260, 263, 511, 514])
def test_strips_that_end_inside_a_quad(proj, kh, kw, w):
    _check(proj, kh, kw, 61, w)


@pytest.mark.parametrize("proj,kh,kw,w", [("FBS", 3, 1, 1), ("FBS", 12, 1, 2), ("FBS", 1, 2, 3), ("FBS", 13, 3, 3), ("BFS", 2, 2, 3), ("BFS", 3, 3, 3),
                                          ("SBM", 2, 2, 2), ("SBM", 3, 3, 3)])
def test_fewer_than_four_columns(proj, kh, kw, w):
    _check(proj, kh, kw, 200, w)


@pytest.mark.parametrize("k", [8, 9, 10, 11])
@pytest.mark.parametrize("w", [11, 12, 255, 256, 257, 263, 264, 265, 266, 267, 268, 269, 511, 512, 520, 522, 523, 524, 700, 1500])
def test_bfs_strips_with_and_without_a_halo(k, w):
    """Last strips with all their 256 columns, with fewer, and ones before them whose halo ends inside a quad."""
    _check("BFS", k, k, 61, w)
