"""The split matrix-core kernel behind AUTO: filters and images at the edges of its strips (240 columns), chunks (16 rows)
and row blocks, and the inputs that its three-part split does not carry.

Every filter below is one that AUTO sends to the kernel at any image size (or, where said, from the size used on).
Tolerance: the split is exact, six of nine products are kept and accumulated in fp32; the parity metric's 1e-5 covers
225 roundings of 2^-24 (1.3e-5 would need them all worst and of one sign).  Integers whose products and sums stay below
2^24 need one part each and come out bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import ORACLE_THREADS, TOL, dev, err2d, run2d
from paper_2010_15884_amd import binding as B

pytestmark = pytest.mark.gpu

# one filter for each number of units, both operand shapes
FILTERS = [(4, 13), (5, 13), (7, 12), (9, 13), (10, 12), (13, 13), (12, 12), (9, 14), (11, 15), (13, 14), (15, 15), (14, 11)]


def _case(h, w, kh, kw, seed=0, top=1.0):
    rng = np.random.default_rng(1000 * kh + kw + seed)
    return rng.uniform(0, top, (h, w)).astype(np.float32), rng.uniform(-1, 1, (kh, kw)).astype(np.float32)


@pytest.mark.parametrize("kh,kw", FILTERS)
@pytest.mark.parametrize("oh,ow", [(1, 1), (16, 240), (17, 241), (15, 243), (33, 482), (100, 719)])
def test_edges_of_strips_and_chunks(kh, kw, oh, ow):
    x, f = _case(oh + kh - 1, ow + kw - 1, kh, kw, top=255.0)
    assert err2d(run2d(x, f, "AUTO"), x, f) <= TOL


@pytest.mark.parametrize("kh,kw", [(9, 13), (13, 13), (15, 15)])
@pytest.mark.parametrize("h", [5000, 8000, 10500, 13001])      # row blocks of 2 .. 5 chunks: odd and even, whole and cut
def test_row_blocks_of_several_chunks(kh, kw, h):
    x, f = _case(h, 600, kh, kw)
    assert err2d(run2d(x, f, "AUTO"), x, f) <= TOL


@pytest.mark.parametrize("kh,kw,h,w", [(13, 13, 60, 500), (15, 15, 60, 500), (11, 11, 1500, 1700)])
def test_integers_exact_and_nothing_written_outside(kh, kw, h, w):
    rng = np.random.default_rng(7)
    x = rng.integers(-100, 100, (h, w)).astype(np.float32)
    f = rng.integers(-9, 9, (kh, kw)).astype(np.float32)
    oh, ow = h - kh + 1, w - kw + 1
    ybig = torch.full((oh + 2, ow + 5), float("nan"), dtype=torch.float32, device="cuda")
    xbig = torch.full((h + 2, w + 7), float("nan"), dtype=torch.float32, device="cuda")      # NaN around the image
    xbig[1:1 + h, 3:3 + w] = dev(x)
    B.sys_conv2d(xbig[1:1 + h, 3:3 + w], f, ybig[1:1 + oh, 1:1 + ow])
    torch.cuda.synchronize()
    out = ybig.cpu().numpy()
    assert np.array_equal(out[1:1 + oh, 1:1 + ow], oracle.conv2d(x, f, ORACLE_THREADS).astype(np.float32))
    out[1:1 + oh, 1:1 + ow] = np.nan
    assert np.isnan(out).all()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 1e30, -3e38, 1e-20, 1e-39])
@pytest.mark.parametrize("kh,kw,h,w", [(9, 13, 70, 500), (13, 13, 8000, 600), (15, 15, 8000, 600)])
def test_values_the_split_does_not_carry(value, kh, kw, h, w):
    """The explicit FBS projection gives what such a value makes of the outputs whose window holds it, and of no others."""
    x, f = _case(h, w, kh, kw, seed=3)
    for r, c in [(0, 0), (15, 239), (16, 240), (47, 256), (h - 1, w - 1), (h // 2, 3)]:
        x[r, c] = value
    d = dev(x)
    want, got = B.sys_conv2d(d, f, projection="FBS"), B.sys_conv2d(d, f)
    assert torch.equal(torch.isnan(want), torch.isnan(got)) and torch.equal(torch.isinf(want), torch.isinf(got))
    ok = torch.isfinite(want)
    scale = B.sys_conv2d(d.abs(), np.abs(f), projection="FBS")[ok]
    assert ((want[ok] - got[ok]).abs() <= TOL * scale).all()


def test_small_numbers_keep_their_precision():
    x, f = _case(80, 500, 13, 13, seed=4)
    for s in (1e-9, 1e-15, 1e-30, 1e15, 1e25):
        xs = (x * s).astype(np.float32)
        assert err2d(run2d(xs, f, "AUTO"), xs, f) <= TOL


@pytest.mark.parametrize("tap", [1e-25, 1e20, np.inf, np.nan])
def test_taps_outside_the_range_take_the_general_path(tap):
    x, f = _case(80, 500, 13, 13, seed=5)
    f[3, 4] = tap
    d = dev(x)
    a, b = B.sys_conv2d(d, f), B.sys_conv2d(d, f, projection="FBS")
    assert torch.equal(a.nan_to_num(nan=1.0), b.nan_to_num(nan=1.0)) and torch.equal(torch.isnan(a), torch.isnan(b))


def test_replayed_from_a_graph():
    x, f = _case(300, 700, 13, 13, seed=6)
    d = dev(x)
    y = torch.empty(288, 688, dtype=torch.float32, device="cuda")
    want = B.sys_conv2d(d, f).clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.sys_conv2d(d, f, y)
    for _ in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
