"""The images of the GPU tests of the stride-2 strips reach every kernel that the launcher can take (its own rule, host code without a GPU)."""
import ctypes

from paper_2010_15884_amd import binding as B
from test_gpu_stride2_2d import STRIP_IMAGES, STRIPS


def test_gpu_tests_reach_every_strip_kernel():
    rows = B.lib()["_ZN7sysconv25conv2d_stride2_strip_rowsEiiii"]
    rows.argtypes, rows.restype = [ctypes.c_int] * 4, ctypes.c_int
    taken = {(kw, rows((h - kh) // 2 + 1, (w - kw) // 2 + 1, kh, kw)) for kh, kw in STRIPS if kh != kw or kh == 1 or kh > 5 for h, w in STRIP_IMAGES}
    assert taken == {(kw, 1) for kw in range(1, 16)} | {(kw, 2) for kw in range(1, 16)} | {(kw, 3) for kw in range(2, 12)}
