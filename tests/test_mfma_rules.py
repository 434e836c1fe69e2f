"""The images of the GPU tests of the MFMA projection reach both kernels for every number of units, with blocks that end everywhere in a chunk (host code without a GPU)."""
import ctypes

from paper_2010_15884_amd import binding as B
from test_gpu_mfma import LDS_IMAGES, WIDE_PITCH


def _host(mangled, args, restype):
    fn = B.lib()[mangled]
    fn.argtypes, fn.restype = args, restype
    return fn


def _units(kh):
    return (kh + 4) // 2


def test_results_through_lds_for_every_number_of_units():
    i, z = ctypes.c_int, ctypes.c_size_t
    rows_out = _host("_ZN7sysconv20conv2d_mfma_rows_outEiim", [i, i, z], ctypes.c_bool)
    block_rows = _host("_ZN7sysconv22conv2d_mfma_block_rowsEiimi", [i, i, z, i], i)
    ends = {}
    for kh, kw, h, w in LDS_IMAGES:
        oh, ow = h - kh + 1, w - kw + 1
        rows = block_rows(oh, ow, ow, kh)
        assert rows_out(oh, ow, ow) and ow % 240 and rows < oh and oh % rows % 16, (kh, kw)       # a cut strip, several blocks, a last one that ends inside a chunk
        ends.setdefault(_units(kh), set()).add(rows % 16)
    assert sorted(ends) == [2, 3, 4, 5, 6, 7, 8] and all(e - {0} for e in ends.values())          # as the others do
    assert set().union(*ends.values()) >= {4, 8, 12}
    assert {_units(kh) for kh, _ in WIDE_PITCH} == set(range(2, 9)) and rows_out(12, 491, (1 << 25) + 8) and not rows_out(12, 491, 1 << 25)
    assert not rows_out(6300, 6300, 6300) and rows_out(6400, 6400, 6400)
