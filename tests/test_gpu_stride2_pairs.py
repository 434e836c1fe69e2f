"""The stride-2 strips of two outputs a lane (conv2d_fbs_stride2_pair_kernel): every width with every number of rows, into a pitched output whose surroundings
stay untouched, from a region of a wider image of NaN.  test_stride2_pair_rules.py checks without a GPU that these images reach all kernels."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import ORACLE_THREADS, TOL, dev
from paper_2010_15884_amd import binding as B
from paper_2010_15884_amd import workloads as W

pytestmark = pytest.mark.gpu

# heights odd and even, below and above the widths; one strip and a cut one (145 of 120 to 128 columns), wavefronts of one row 1400 .. 46002
FILTERS = [(5, 1), (3, 2), (7, 3), (9, 4), (3, 5), (7, 6), (7, 7), (9, 8), (9, 9), (5, 10), (11, 11), (12, 12), (2, 13), (6, 14), (15, 15), (6, 7), (14, 3)]
OUTPUTS = [(701, 145), (4001, 145), (9002, 145), (23001, 145)]


# more than 70000 wavefronts of one row: the strips of four outputs a lane, three rows each (whole, one and two left over), strips of 252 columns inside and at the edge
LARGE_TWO_COLUMNS = [(15, 35003, 129), (3, 23400, 258), (8, 7900, 1025)]


def run_in_a_region(kh, kw, h, w):
    oh, ow = (h - kh) // 2 + 1, (w - kw) // 2 + 1
    x, f = W.random_case(kh * 100 + kw, (h, w), (kh, kw), x_range=(0.0, 1.0))
    big = torch.full((h, w + 5), float("nan"), dtype=torch.float32, device="cuda")
    big[:, 2:2 + w] = dev(x)
    out = torch.full((oh + 2, ow + 3), float("nan"), dtype=torch.float32, device="cuda")
    B.sys_conv2d_strided(big[:, 2:2 + w], f, 2, out[1:1 + oh, 1:1 + ow])
    torch.cuda.synchronize()
    y = out.cpu().numpy()
    ref = oracle.conv2d_strided(x, f, 2, ORACLE_THREADS)
    scale = oracle.absdot2d_strided(x, f, 2, ORACLE_THREADS)
    assert oracle.max_rel_err(np.ascontiguousarray(y[1:1 + oh, 1:1 + ow]), ref, scale) <= TOL
    y[1:1 + oh, 1:1 + ow] = np.nan
    assert np.isnan(y).all()


@pytest.mark.parametrize("kh,kw", FILTERS)
@pytest.mark.parametrize("oh,ow", OUTPUTS)
def test_every_width_and_number_of_rows(kh, kw, oh, ow):
    run_in_a_region(kh, kw, 2 * (oh - 1) + kh + (kw & 1), 2 * (ow - 1) + kw + (kh & 1))


@pytest.mark.parametrize("kh,oh,ow", LARGE_TWO_COLUMNS)
def test_two_columns_on_large_images(kh, oh, ow):
    run_in_a_region(kh, 2, 2 * (oh - 1) + kh, 2 * (ow - 1) + 2 + (kh & 1))
