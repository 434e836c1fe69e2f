"""The images of the GPU tests of the stride-2 strips of four outputs a lane reach every kernel that the launcher can take (its own rules, host code without a GPU)."""
import ctypes

from paper_2010_15884_amd import binding as B
from test_gpu_stride2_pairs import LARGE_TWO_COLUMNS
from test_gpu_stride2_strips import NARROW, NARROW_ROWS, SINGLE_ROW_IMAGES


def _host(name, n, restype):
    fn = B.lib()[f"_ZN7sysconv{len(name)}{name}E" + "i" * n]
    fn.argtypes, fn.restype = [ctypes.c_int] * n, restype
    return fn


def test_gpu_tests_reach_every_strip_kernel():
    takes, rows = _host("conv2d_stride2_takes_strips", 5, ctypes.c_bool), _host("conv2d_stride2_strip_rows", 4, ctypes.c_int)
    calls = [(w, (h - 1) // 2 + 1, (w - kw) // 2 + 1, 1, kw) for kw in range(1, 16) for h, w in SINGLE_ROW_IMAGES]
    calls += [(w, oh, (w - kw) // 2 + 1, kh, kw) for w, kh, kw in NARROW for oh in NARROW_ROWS]
    calls += [(2 * ow, oh, ow, kh, 2) for kh, oh, ow in LARGE_TWO_COLUMNS]
    assert all(takes(*c) for c in calls)
    taken = {(kw, rows(w, oh, kh, kw), w < 4) for w, oh, ow, kh, kw in calls}
    assert taken == {(kw, 1, False) for kw in range(1, 16)} | {(2, 3, False)} | {(kw, r, True) for kw in (1, 2, 3) for r in (1, 2, 3)}
