"""The FBS strips of 8 to 15 columns (conv2d_fbs_strip_kernel): every width with every number of rows, into a pitched output whose surroundings stay untouched, from a
region of a wider image of NaN, and against the same sums in integers.  test_fbs_strip_rules.py checks without a GPU that these images reach all kernels."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import TOL, dev, err2d
from paper_2010_15884_amd import binding as B
from paper_2010_15884_amd import workloads as W

pytestmark = pytest.mark.gpu

# rows of 12 taps and more, and 7x14 and 7x15, come here from 2 M outputs on; one whole strip (208 .. 244 columns) and a cut one
FILTERS = [(10, 8), (8, 8), (9, 9), (13, 10), (11, 11), (12, 12), (8, 13), (9, 14), (15, 15), (1, 12), (1, 13), (1, 14), (1, 15), (7, 14), (7, 15), (15, 9)]
OUTPUTS = [(701, 301), (3002, 301), (8001, 301)]


@pytest.mark.parametrize("kh,kw", FILTERS)
@pytest.mark.parametrize("oh,ow", OUTPUTS + [(1, 1), (5, 250), (17, 1000)])
def test_every_width_and_number_of_rows(kh, kw, oh, ow):
    h, w = oh + kh - 1, ow + kw - 1
    x, f = W.random_case(kh * 100 + kw, (h, w), (kh, kw), x_range=(0.0, 1.0))
    big = torch.full((h, w + 5), float("nan"), dtype=torch.float32, device="cuda")
    big[:, 2:2 + w] = dev(x)
    out = torch.full((oh + 2, ow + 3), float("nan"), dtype=torch.float32, device="cuda")
    B.sys_conv2d(big[:, 2:2 + w], f, out[1:1 + oh, 1:1 + ow], projection="FBS")
    torch.cuda.synchronize()
    y = out.cpu().numpy()
    assert err2d(np.ascontiguousarray(y[1:1 + oh, 1:1 + ow]), x, f) <= TOL
    y[1:1 + oh, 1:1 + ow] = np.nan
    assert np.isnan(y).all()


@pytest.mark.parametrize("h,w", [(1, 1), (3, 2), (40, 3), (70, 515)])
def test_one_tap(h, w):
    x, f = W.integer_case(h + w, (h, w), (1, 1), x_max=9, w_max=5)
    y = B.sys_conv2d(dev(x), f, projection="FBS")
    assert np.array_equal(y.cpu().numpy().astype(np.float64), oracle.conv2d(x, f))
