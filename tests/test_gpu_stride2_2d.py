"""GPU parity of the stride-2 2-D FBS kernel against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import ORACLE_THREADS, TOL, dev
from paper_2010_15884_amd import binding as B
from paper_2010_15884_amd import workloads as W

pytestmark = pytest.mark.gpu

KSHAPES = [(1, 1), (1, 2), (2, 1), (2, 2), (3, 3), (4, 4), (5, 5), (6, 6), (7, 7), (8, 8), (9, 9), (11, 11), (15, 15),
           (3, 8), (8, 3), (1, 15), (15, 1), (4, 13)]


def run(x, f, proj="FBS"):
    y = B.sys_conv2d_strided(dev(x), f, 2, projection=proj)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def err(y, x, f):
    ref = oracle.conv2d_strided(x, f, 2, ORACLE_THREADS)
    scale = oracle.absdot2d_strided(x, f, 2, ORACLE_THREADS)
    return oracle.max_rel_err(y, ref, scale)


def _images(kh, kw):
    cols = 4 * (64 - ((kw + 1) // 2 + 2) // 4)           # output columns of a tile
    cand = [(kh, kw), (kh + 1, kw + 1), (kh + 2, kw + 3), (41, 301), (40, 300), (2 * 8 + kh - 2, 2 * cols + kw - 2),
            (2 * 8 + kh - 1, 2 * cols + kw - 1), (2 * 8 + kh, 2 * cols + kw), (2 * 17 + kh, 4 * cols + kw + 7), (259, 1533)]
    return [(h, w) for h, w in cand if h >= kh and w >= kw]


@pytest.mark.parametrize("proj", ["FBS", "AUTO"])
@pytest.mark.parametrize("kshape", KSHAPES)
def test_stride2_2d_random_all_sizes(kshape, proj):
    kh, kw = kshape
    for (h, w) in _images(kh, kw):
        x, f = W.random_case(h * 1000 + w + kh, (h, w), (kh, kw), x_range=(0.0, 1.0))
        y = run(x, f, proj)
        assert y.shape == ((h - kh) // 2 + 1, (w - kw) // 2 + 1)
        e = err(y, x, f)
        assert e <= TOL, f"{kh}x{kw} image {h}x{w}: rel err {e}"


@pytest.mark.parametrize("kshape", [(2, 2), (3, 3), (5, 5), (11, 11), (4, 7)])
def test_stride2_2d_integer_data_is_bit_exact(kshape):
    kh, kw = kshape
    for shape in [(150, 700), (151, 701), (33, 1100)]:
        x, f = W.integer_case(kh * 31 + kw + shape[0], shape, (kh, kw), x_max=9, w_max=5)
        y = run(x, f)
        assert np.array_equal(y.astype(np.float64), oracle.conv2d_strided(x, f, 2)), f"{kh}x{kw} {shape}"


def test_stride2_2d_delta_filter_picks_every_second_pixel():
    x, _ = W.random_case(6, (91, 603), (1, 1), x_range=(0.0, 1.0))
    for (kh, kw, p, q) in [(1, 1, 0, 0), (3, 3, 2, 1), (5, 5, 0, 4), (5, 5, 4, 3), (11, 11, 10, 10), (4, 7, 3, 0), (2, 15, 1, 14)]:
        f = np.zeros((kh, kw), np.float32)
        f[p, q] = 1.0
        y = run(x, f)
        assert np.array_equal(y, x[p:p + 2 * y.shape[0]:2, q:q + 2 * y.shape[1]:2]), (kh, kw, p, q)


def test_stride2_2d_is_every_second_output_of_stride1_on_integer_data():
    x, f = W.integer_case(77, (300, 900), (5, 5), x_max=9, w_max=5)
    y2 = run(x, f)
    y1 = B.sys_conv2d(dev(x), f, projection="FBS").cpu().numpy()
    assert np.array_equal(y2, y1[::2, ::2])


def test_stride1_through_the_strided_entry_is_sys_conv2d():
    x, f = W.random_case(3, (200, 500), (5, 5), x_range=(0.0, 1.0))
    for proj in ("AUTO", "FBS", "SBM", "BFS"):
        a = B.sys_conv2d_strided(dev(x), f, 1, projection=proj).cpu().numpy()
        b = B.sys_conv2d(dev(x), f, projection=proj).cpu().numpy()
        assert np.array_equal(a, b), proj


def test_stride2_2d_pitched_views_and_guard_bands():
    for (kh, kw) in [(3, 3), (5, 5), (6, 2)]:
        h, w = 61, 1047
        x, f = W.random_case(9 + kh, (h, w), (kh, kw), x_range=(0.0, 1.0))
        xbig = torch.zeros((h + 2, w + 13), dtype=torch.float32, device="cuda")
        xbig[1:1 + h, 5:5 + w] = dev(x)
        oh, ow = (h - kh) // 2 + 1, (w - kw) // 2 + 1
        ybig = torch.full((oh + 4, ow + 11), float("nan"), dtype=torch.float32, device="cuda")
        B.sys_conv2d_strided(xbig[1:1 + h, 5:5 + w], f, 2, ybig[2:2 + oh, 3:3 + ow], projection="FBS")
        torch.cuda.synchronize()
        out = ybig.cpu().numpy()
        inner = out[2:2 + oh, 3:3 + ow].copy()
        out[2:2 + oh, 3:3 + ow] = np.nan
        assert np.isnan(out).all(), f"{kh}x{kw} wrote outside its output window"
        assert err(inner, x, f) <= TOL, f"{kh}x{kw}"


@pytest.mark.parametrize("seed", range(16))
def test_stride2_2d_random_shapes(seed):
    rng = np.random.default_rng(12000 + seed)
    kh, kw = int(rng.integers(1, 16)), int(rng.integers(1, 16))
    if seed % 4 == 0:                                          # long rows: the banded work order
        h, w = kh + int(rng.integers(0, 40)), max(8192, kw) + int(rng.integers(0, 3000))
    else:
        h, w = kh + int(rng.integers(0, 300)), kw + int(rng.integers(0, 1500))
    x, f = W.random_case(300 + seed, (h, w), (kh, kw), x_range=(0.0, 1.0))
    e = err(run(x, f), x, f)
    assert e <= TOL, f"seed {seed} {kh}x{kw} image {h}x{w}: rel err {e}"


def test_stride2_2d_unsupported_requests_launch_nothing():
    x = torch.zeros((100, 100), dtype=torch.float32, device="cuda")
    y = torch.full((60, 60), 7.0, dtype=torch.float32, device="cuda")
    f = np.ones((5, 5), np.float32)
    for proj, stride in [("SBM", 2), ("BFS", 2), ("FBS", 3), ("AUTO", 4)]:
        with pytest.raises(B.SysconvError) as e:
            B.sys_conv2d_strided(x, f, stride, y, projection=proj)
        assert e.value.status == B.SYS_ERR_UNSUPPORTED
    with pytest.raises(B.SysconvError) as e:
        B.sys_conv2d_strided(x, f, 0, y, projection="FBS")
    assert e.value.status == B.SYS_ERR_SIZE
    torch.cuda.synchronize()
    assert (y == 7.0).all()


# Filters of every width on images that fill the chip and more (which kernels run on them: test_stride2_pair_rules.py and test_stride2_rules.py, for images of their own).
STRIPS = [(15, 1), (1, 1), (9, 2), (13, 3), (3, 4), (4, 5), (1, 6), (6, 6), (7, 7), (2, 8), (9, 9), (5, 10), (4, 11), (11, 11), (2, 12), (3, 13), (6, 14),
          (15, 15)]
STRIP_IMAGES = [(4003, 4099), (2801, 4101), (2401, 2403), (700, 2301)]


@pytest.mark.parametrize("kh,kw", STRIPS)
@pytest.mark.parametrize("h,w", STRIP_IMAGES)
def test_stride2_2d_strips_of_two_and_three_rows(kh, kw, h, w):
    """Whole strips and the cut one at the right edge, into a pitched output whose surroundings stay untouched."""
    x, f = W.random_case(kh * 100 + kw, (h, w), (kh, kw), x_range=(0.0, 1.0))
    oh, ow = (h - kh) // 2 + 1, (w - kw) // 2 + 1
    big = torch.full((oh + 2, ow + 5), float("nan"), dtype=torch.float32, device="cuda")
    B.sys_conv2d_strided(dev(x), f, 2, big[1:1 + oh, 2:2 + ow])
    torch.cuda.synchronize()
    out = big.cpu().numpy()
    assert err(np.ascontiguousarray(out[1:1 + oh, 2:2 + ow]), x, f) <= TOL
    out[1:1 + oh, 2:2 + ow] = np.nan
    assert np.isnan(out).all()


@pytest.mark.parametrize("kh,kw", [(6, 6), (13, 3), (15, 15), (15, 1), (2, 2), (4, 4)])
@pytest.mark.parametrize("h,w", [(4003, 4099), (2801, 4101), (2401, 2403), (700, 1301)])
def test_stride2_2d_strips_keep_infinities_in_their_windows(kh, kw, h, w):
    x, f = W.random_case(kh, (h, w), (kh, kw), x_range=(0.0, 1.0))
    bad = [(0, 0), (h - 1, w - 1), (350, 511), (351, 512)]
    for r, c in bad:
        x[r, c] = np.inf
    y = run(x, f)
    want = np.zeros(y.shape, bool)
    for r, c in bad:
        rr, cc = np.arange(y.shape[0]) * 2, np.arange(y.shape[1]) * 2
        want |= np.outer((rr <= r) & (r < rr + kh), (cc <= c) & (c < cc + kw))
    assert np.array_equal(~np.isfinite(y), want)


@pytest.mark.parametrize("w", [200, 257, 505, 508, 511, 512, 513, 761, 1016, 1300])
def test_stride2_2d_2x2_right_hand_strip(w):
    """The last strip of 2x2 filters, which loads its lanes straight where the others exchange (504 input columns a strip)."""
    x, f = W.random_case(w, (41, w), (2, 2), x_range=(0.0, 1.0))
    assert err(run(x, f), x, f) <= TOL


# One-row and two-row wavefronts on either side of both lines (3000 and 4096 wavefronts of one row; strips of 248 to 252 outputs), the
# single-row filter, and right-hand strips that end inside a lane's quad, with one whole strip and without.
@pytest.mark.parametrize("kh,kw,oh,ow", [(4, 6, 2900, 200), (4, 6, 3100, 200), (9, 9, 4090, 130), (9, 9, 4102, 130), (1, 7, 5000, 90), (2, 1, 1501, 505),
                                         (12, 12, 40, 253), (3, 5, 77, 250), (6, 6, 33, 1)])
@pytest.mark.parametrize("extra", [0, 1])                       # an odd and an even number of columns
def test_stride2_2d_rows_of_a_wavefront_and_right_edge(kh, kw, oh, ow, extra):
    h, w = 2 * (oh - 1) + kh, 2 * (ow - 1) + kw + extra
    x, f = W.random_case(kh * 100 + kw + extra, (h, w), (kh, kw), x_range=(0.0, 1.0))
    big = torch.full((h, w + 9), float("nan"), dtype=torch.float32, device="cuda")     # a region of a wider image of NaN
    big[:, :w] = dev(x)
    y = B.sys_conv2d_strided(big[:, :w], f, 2)
    torch.cuda.synchronize()
    assert err(y.cpu().numpy(), x, f) <= TOL


@pytest.mark.parametrize("kh,kw,w", [(2, 1, 1), (5, 1, 2), (2, 2, 2), (2, 2, 3), (7, 2, 3), (3, 3, 3), (15, 3, 3)])
@pytest.mark.parametrize("h", [20, 9001])
def test_stride2_2d_images_of_fewer_than_four_columns(kh, kw, w, h):
    x, f = W.random_case(kh * 10 + kw, (h, w), (kh, kw), x_range=(0.0, 1.0))
    y = B.sys_conv2d_strided(dev(x), f, 2)
    torch.cuda.synchronize()
    assert err(y.cpu().numpy(), x, f) <= TOL
