"""AUTO against the projections by name for small square filters.  SBM adds an output's taps in an order of its own, so its bits tell it from the
others; FBS and BFS share theirs, and which of these two AUTO takes on either side of its lines is pinned on the host function that chooses
(abi_san_driver.cpp).
"""
import pytest
import torch

from gpu_common import dev
from paper_2010_15884_amd import binding as B
from paper_2010_15884_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,k,proj", [
    (300, 1024, 5, "BFS"), (300, 1000, 5, "FBS"),                      # power-of-two pitch or not
    (700, 4096, 2, "BFS"), (700, 4096, 3, "BFS"), (800, 4096, 5, "BFS"),
    (1024, 1024, 6, "BFS"), (1600, 1024, 6, "BFS"), (4096, 2048, 6, "BFS"),
    (300, 2048, 7, "FBS"), (1024, 1024, 7, "BFS"), (7800, 2048, 7, "BFS"), (8200, 2048, 7, "SBM"),
    (700, 4096, 7, "FBS"), (800, 4096, 7, "SBM"), (1700, 1701, 7, "FBS"), (1800, 1801, 7, "SBM"),
    (300, 300, 8, "SBM"), (300, 300, 6, "FBS"),
])
def test_auto_takes(h, w, k, proj):
    x, f = W.random_case(h + w + k, (h, w), (k, k), x_range=(0.0, 255.0))
    d = dev(x)
    auto = B.sys_conv2d(d, f)
    assert torch.equal(auto, B.sys_conv2d(d, f, projection=proj))
    for other in ("FBS", "BFS", "SBM"):
        if (other == "SBM") != (proj == "SBM"):
            assert not torch.equal(auto, B.sys_conv2d(d, f, projection=other))
