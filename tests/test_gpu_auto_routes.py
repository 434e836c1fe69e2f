"""Which kernel AUTO takes on either side of its lines for small square filters: its bits are those of the projection named there (the
kernels add an output's taps in different orders, so another one's bits differ somewhere)."""
import pytest
import torch

from gpu_common import dev
from paper_2010_15884_amd import binding as B
from paper_2010_15884_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,k,proj", [
    (300, 1024, 5, "BFS"), (300, 1000, 5, "FBS"),                      # power-of-two pitch or not
    (700, 4096, 2, "BFS"), (700, 4096, 3, "FBS"), (800, 4096, 5, "BFS"),       # 16 KB rows: 3 M outputs
    (1024, 1024, 6, "BFS"), (1600, 1024, 6, "FBS"), (4096, 2048, 6, "BFS"),    # 6x6: 1.5 M and 8 M
    (300, 2048, 7, "BFS"), (700, 4096, 7, "FBS"), (800, 4096, 7, "SBM"), (1700, 1701, 7, "FBS"), (1800, 1801, 7, "SBM"),
    (300, 300, 8, "SBM"), (300, 300, 6, "FBS"),
])
def test_auto_takes(h, w, k, proj):
    x, f = W.random_case(h + w + k, (h, w), (k, k), x_range=(0.0, 255.0))
    d = dev(x)
    auto = B.sys_conv2d(d, f)
    assert torch.equal(auto, B.sys_conv2d(d, f, projection=proj))
    for other in ("FBS", "BFS", "SBM"):
        if other == "SBM" and proj != "SBM" or proj == "SBM" and other != "SBM":
            assert not torch.equal(auto, B.sys_conv2d(d, f, projection=other))      # (FBS and BFS share an order)
