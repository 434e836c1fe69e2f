"""The images of the GPU tests of the FBS strips reach every kernel that the launcher can take, and its lines (host code without a GPU)."""
import ctypes

from paper_2010_15884_amd import binding as B
from test_gpu_fbs_strips import FILTERS, OUTPUTS


def _host(name, n, restype):
    fn = B.lib()[f"_ZN7sysconv{len(name)}{name}E" + "i" * n]
    fn.argtypes, fn.restype = [ctypes.c_int] * n, restype
    return fn


def test_gpu_tests_reach_every_strip_kernel():
    rows, tiles = _host("conv2d_fbs_strip_rows", 4, ctypes.c_int), _host("conv2d_fbs_static_serves", 4, ctypes.c_bool)
    taken = {(kw, rows(oh, ow, kh, kw)) for kh, kw in FILTERS for oh, ow in OUTPUTS if not tiles(oh, ow, kh, kw)}
    assert taken == {(kw, r) for kw in range(8, 16) for r in (1, 2, 3)} | {(kw, 4) for kw in range(12, 16)}


def test_lines():
    rows, tiles = _host("conv2d_fbs_strip_rows", 4, ctypes.c_int), _host("conv2d_fbs_static_serves", 4, ctypes.c_bool)
    for line, below, above in ((4000, 1, 2), (15000, 2, 3)):
        assert rows(line, 244, 11, 11) == below and rows(line + 1, 244, 11, 11) == above and rows(line // 2 + 1, 245, 11, 11) == above
    for kh in range(1, 16):
        for kw in range(1, 16):
            few, many = tiles(1000, 2000, kh, kw), tiles(1001, 2000, kh, kw)
            assert few == (min(kh, kw) <= 7)
            assert many == (few and not (kh == 1 and kw >= 12) and not (kh == 7 and kw >= 14))


def test_auto_line_to_the_strips():
    fn = B.lib()["_ZN7sysconv24conv2d_vector_projectionEiimii"]
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_int, ctypes.c_int], ctypes.c_int
    for pitch in (1000, 1024):
        for k in (9, 10, 11):
            assert fn(400, 1000, pitch, k, k) == B.SYS_PROJ_FBS and fn(1, 1, pitch, k, k) == B.SYS_PROJ_FBS
            assert fn(401, 1000, pitch, k, k) == B.SYS_PROJ_SBM
            assert fn(3000, 100, pitch, k, k) == B.SYS_PROJ_FBS and fn(3001, 100, pitch, k, k) == B.SYS_PROJ_SBM
        assert fn(300, 300, pitch, 8, 8) == B.SYS_PROJ_SBM
