"""Which calls AUTO sends to the split matrix-core kernel (the library's own rule, host code without a GPU)."""
import ctypes

import pytest

from paper_2010_15884_amd import binding as B
from test_gpu_split import CUT_CHUNKS, EDGES, FILTERS, MARKED_IMAGES, SEVERAL_CHUNKS


def split_pays(oh, ow, kh, kw):
    fn = B.lib()["_ZN7sysconv17conv2d_split_paysEiiii"]
    fn.argtypes, fn.restype = [ctypes.c_int] * 4, ctypes.c_bool
    return fn(oh, ow, kh, kw)


# The split's sums are two to four times as exact as the vector kernels', and a caller of AUTO has no say in it: filters that it serves from a size on
# keep it from there on, also on sizes where a vector kernel is a little quicker.
@pytest.mark.parametrize("kh,kw,least", [(4, 12, 1), (4, 13, 1), (5, 12, 1), (5, 13, 1), (6, 12, 1), (6, 13, 1), (7, 12, 1), (7, 13, 1), (6, 14, 1), (6, 15, 1),
                                         (7, 14, 1), (7, 15, 1), (3, 12, 2236), (3, 13, 2236), (12, 6, 1440), (12, 7, 1420), (13, 5, 1900), (13, 6, 1420), (13, 7, 1420),
                                         (8, 9, 1), (9, 8, 1), (10, 9, 1), (12, 9, 1), (15, 15, 1), (14, 11, 1)])
def test_filters_keep_the_kernel_with_the_smaller_error(kh, kw, least):
    for s in (1, 17, 100, 277, 317, 500, 700, 900, 1100, 1300, 1600, 2100, 2400, 3000, 4096, 8192):
        if s >= least:
            assert split_pays(s, s, kh, kw), s


# What the strips of 240 columns and the chunks of 16 rows compute for padding counts in full where the two kernels are close: the first is level or slower on the split
# (measured 1.04 .. 1.2 times the vector kernel), the second (no padding) faster.
@pytest.mark.parametrize("kh,kw,padded,even", [(10, 10, (2046, 1002), (2046, 1200)), (5, 9, (7737, 723), (7737, 720)), (7, 8, (6757, 721), (6757, 720)),
                                               (6, 8, (6483, 1203), (6480, 1440)), (7, 9, (1607, 1700), (2400, 1920)), (9, 6, (4591, 1926), (4592, 1920)),
                                               (7, 11, (737, 850), (1280, 960)), (5, 11, (508, 4639), (1200, 2400)), (10, 6, (6129, 1483), (6128, 1440))])
def test_padding_counts_in_full(kh, kw, padded, even):
    assert not split_pays(*padded, kh, kw)
    assert split_pays(*even, kh, kw)


def block_rows(oh, ow, kh, kw):
    fn = B.lib()["_ZN7sysconv23conv2d_split_block_rowsEiiii"]
    fn.argtypes, fn.restype = [ctypes.c_int] * 4, ctypes.c_int
    return fn(oh, ow, kh, kw)


def test_calls_of_the_gpu_tests_run_the_split_kernel():
    for kh, kw in FILTERS:
        assert all(split_pays(oh, ow, kh, kw) for oh, ow in EDGES)
    for kh, kw in [(9, 13), (13, 13), (15, 15), (6, 14)]:
        assert all(split_pays(h - kh + 1, 601 - kw, kh, kw) for h in SEVERAL_CHUNKS + CUT_CHUNKS)
    for kh, kw, h, w in [(13, 13, 60, 500), (15, 15, 60, 500), (11, 11, 1500, 1700), (9, 13, 70, 500), (13, 13, 8000, 600), (15, 15, 8000, 600), (9, 13, 300, 700),
                         (13, 13, 150, 500), (15, 15, 150, 500), (13, 13, 80, 500), (13, 13, 300, 700), *MARKED_IMAGES]:
        assert split_pays(h - kh + 1, w - kw + 1, kh, kw), (kh, kw, h, w)


def test_blocks_of_the_gpu_tests_end_everywhere_in_a_chunk():
    for kh, kw, rows in [(9, 13, 4), (13, 13, 4), (15, 15, 8), (6, 14, 8)]:
        assert [block_rows(h - kh + 1, 601 - kw, kh, kw) for h in SEVERAL_CHUNKS] == [32, 48, 64, 80]
        assert {block_rows(h - kh + 1, 601 - kw, kh, kw) // rows % (16 // rows) for h in CUT_CHUNKS + SEVERAL_CHUNKS} == set(range(16 // rows))


def test_images_with_marked_chunks_have_blocks_of_every_length():
    """Chunks (16 rows) of a row block on the images of the GPU test: the first mark word alone, both, and the most there can be."""

    def chunks(kh, kw, h, w):
        return -(-block_rows(h - kh + 1, w - kw + 1, kh, kw) // 16)

    assert [chunks(*i) for i in MARKED_IMAGES] == [1, 2, 12, 12, 14, 32, 48, 56]
    # no image has longer blocks: what the marks have room for, with the chunk that only finishes groups
    for kh, kw, most in ((13, 13, 32), (4, 13, 32), (15, 15, 56), (6, 14, 56)):
        seen = {chunks(kh, kw, h, w) for w in (100, 250, 600, 1201, 5000, 40000) for h in range(1000, 200000, 500)}
        assert max(seen) == most


@pytest.mark.parametrize("kh,kw,h,w,groups", [(11, 14, 744, 580, 2), (13, 14, 304, 2677, 2), (10, 14, 739, 747, 2), (12, 15, 1473, 288, 2),      # one group: more than 256 workgroups
                                              (14, 14, 500, 500, 1), (15, 15, 300, 400, 1), (9, 15, 282, 797, 1)])
def test_eight_by_two_prefers_one_workgroup_a_cu(kh, kw, h, w, groups):
    """Blocks of one group, two a CU, are 10 % slower than blocks of two groups, one a CU; one a CU they are 6 to 8 % faster."""
    assert block_rows(h - kh + 1, w - kw + 1, kh, kw) == 8 * groups
