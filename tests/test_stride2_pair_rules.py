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
    assert taken == ({(kw, r) for kw in range(1, 16) for r in (1, 2)} | {(kw, 3) for kw in range(1, 16) if kw not in (10, 11)} | {(kw, 4) for kw in range(4, 12)})


def test_lines():
    rows = _rows()
    for strips in (1, 2):                                      # columns a strip: 124 at a width of 7, 118 at 11, 116 at 12, 126 at 3
        for kh, kw, ow, lines in ((7, 7, 124, [(5000, 1, 2), (11500, 2, 3), (45000, 3, 4)]), (8, 7, 124, [(5000, 1, 2), (11500, 2, 3), (70000, 3, 4)]),
                                  (11, 11, 118, [(5000, 1, 2), (45000, 2, 4)]), (10, 11, 118, [(5000, 1, 2), (45000, 2, 4)]), (12, 12, 116, [(5000, 1, 2), (40000, 2, 3)]),
                                  (5, 3, 126, [(3000, 1, 2), (11500, 2, 3), (32000, 3, 2), (70000, 2, 3)]), (5, 2, 128, [(3000, 1, 2), (11500, 2, 3), (22000, 3, 2), (70000, 2, 3)])):
            for line, below, above in lines:
                assert rows(line // strips, ow * strips, kh, kw) == below and rows(line // strips + 1, ow * strips, kh, kw) == above, (kh, kw, line)
    assert rows(1 << 30, 1 << 30, 15, 15) == 3                 # no overflow


def test_calls_that_more_rows_slowed_down():
    """Images and filters that three or four rows made slower than the strips before (us, those / these / with the rows below)."""
    rows = _rows()
    for h, w, kh, kw, best in ((5767, 5767, 7, 2, 2), (5284, 5284, 12, 1, 2), (3942, 3942, 9, 1, 2),               # 28.7 / 34.8 / 26.3, 27.2 / 32.8 / 26.9, 15.6 / 18.2 / 15.3
                               (7138, 3115, 13, 3, 2), (1984, 5907, 14, 13, 2), (3502, 3502, 10, 10, 2),           # 29.2 / 31.5 / 26.4, 25.5 / 27.4 / 25.0, 19.2 / 20.9 / 19.9
                               (3658, 293, 15, 2, 2), (5109, 507, 14, 14, 2),                               # 5.5 / 6.2 / 5.6, 11.3 / 12.4 / 11.2
                               (6517, 6174, 8, 10, 4), (5413, 5413, 6, 10, 4), (7206, 7206, 8, 8, 4)):             # 46.5 / 49.8 / 44.7, 27.7 / 30.2 / 26.8, 58.1 / 59.5 / 55.7
        assert rows((h - kh) // 2 + 1, (w - kw) // 2 + 1, kh, kw) == best


def test_two_columns_on_large_images_take_the_strips():
    """More than 70000 wavefronts of one row: the pair form is 2 to 23 % slower there with any number of rows."""
    fn = B.lib()["_ZN7sysconv27conv2d_stride2_takes_stripsEiiiii"]
    fn.argtypes, fn.restype = [ctypes.c_int] * 5, ctypes.c_bool
    for oh, ow in ((35000, 129), (35001, 129), (70000, 128), (70001, 1)):
        for kw in (1, 2, 3, 4, 15):
            assert fn(2 * ow + kw + 8, oh, ow, 9, kw) == (kw == 2 and oh in (35001, 70001))
    assert fn(3, 5, 1, 9, 2) and fn(3, 5, 1, 9, 3) and not fn(4, 5, 1, 9, 3) and fn(4000, 5, 2000, 1, 3)
