"""The images of the GPU tests of the stride-2 strips of two outputs a lane reach every kernel that the launcher can take, and its lines (host code without a GPU)."""
import ctypes

from paper_2010_15884_amd import binding as B
from test_gpu_stride2_pairs import FILTERS, OUTPUTS


def _rows():
    rows = B.lib()["_ZN7sysconv24conv2d_stride2_pair_rowsEiiii"]
    rows.argtypes, rows.restype = [ctypes.c_int] * 4, ctypes.c_int
    return rows


def test_gpu_tests_reach_every_pair_kernel():
    rows = _rows()
    taken = {(kw, rows(oh, ow, kh, kw)) for kh, kw in FILTERS if kh != kw or kh > 5 for oh, ow in OUTPUTS}
    assert {(kw, r) for kw in range(1, 16) for r in (1, 2, 3)} <= taken
    assert {(kw, 4) for kw in range(1, 12)} == {t for t in taken if t[1] == 4}


def test_lines():
    rows = _rows()
    for strips in (1, 2):                                      # 124 columns a strip at a width of 7, 116 at 12
        ow7, ow12 = 124 * strips, 116 * strips
        for line, below, above in ((5000, 1, 2), (11500, 2, 3), (45000, 3, 4)):
            assert rows(line // strips, ow7, 7, 7) == below and rows(line // strips + 1, ow7, 7, 7) == above
        assert rows(45001, ow7, 8, 7) == 3                     # an even height
        for line, below, above in ((8500, 1, 2), (20000, 2, 3)):
            assert rows(line // strips, ow12, 12, 12) == below and rows(line // strips + 1, ow12, 12, 12) == above
    assert rows(1 << 30, 1 << 30, 15, 15) == 3                 # no overflow
