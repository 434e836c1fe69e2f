"""The split matrix-core kernel behind AUTO: filters and images at the edges of its strips (240 columns), chunks (16 rows)
and row blocks, and the inputs that its three-part split does not carry.

Every call below is one that AUTO sends to the kernel (test_split_rules.py checks that without a GPU).
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
EDGES = [(1, 1), (16, 240), (17, 241), (15, 243), (33, 482), (100, 719)]                   # outputs
SEVERAL_CHUNKS = [5000, 8000, 10500, 13001]                                               # rows of 600 columns: row blocks of 2 .. 5 chunks, odd and even, whole and cut
CUT_CHUNKS = [900, 2000, 3400, 4100, 5500, 6200, 6900]                                    # blocks of 3, 6, 5, 7, 9, 10, 11 groups (8 x 2: 1 .. 6): chunks cut after each group


def _case(h, w, kh, kw, seed=0, top=1.0):
    rng = np.random.default_rng(1000 * kh + kw + seed)
    return rng.uniform(0, top, (h, w)).astype(np.float32), rng.uniform(-1, 1, (kh, kw)).astype(np.float32)


@pytest.mark.parametrize("kh,kw", FILTERS)
def test_auto_runs_the_split_kernel(kh, kw):
    """Every vector kernel takes an output's taps in an order of its own in fp32; the split's sums round elsewhere.  So on random
    data AUTO's bits differ from those of every projection that could have run instead."""
    x, f = _case(100 + kh - 1, 719 + kw - 1, kh, kw, seed=11, top=255.0)
    d = dev(x)
    auto = B.sys_conv2d(d, f)
    for proj in ("FBS", "SBM", "BFS"):
        if B.sys_conv2d_has(proj, kh, kw):
            assert (auto != B.sys_conv2d(d, f, projection=proj)).float().mean() > 0.2, proj


@pytest.mark.parametrize("kh,kw,oh,ow", [(4, 12, 500, 700), (4, 13, 900, 901), (5, 12, 700, 600), (6, 13, 500, 500), (7, 12, 600, 500), (7, 13, 400, 700),
                                         (13, 5, 1900, 2101), (12, 7, 1500, 1500), (3, 12, 2300, 2301), (10, 8, 500, 700)])
def test_auto_errs_less_than_the_vector_kernels(kh, kw, oh, ow):
    """2-norm of the error against 64 bits: measured 0.22 .. 0.37 of the FBS kernels'."""
    x, f = _case(oh + kh - 1, ow + kw - 1, kh, kw, seed=14)
    ref = oracle.conv2d(x, f, ORACLE_THREADS)
    auto, fbs = (np.linalg.norm(run2d(x, f, p) - ref) for p in ("AUTO", "FBS"))
    assert auto <= 0.5 * fbs, auto / fbs


@pytest.mark.parametrize("kh,kw", FILTERS)
@pytest.mark.parametrize("oh,ow", EDGES)
def test_edges_of_strips_and_chunks(kh, kw, oh, ow):
    x, f = _case(oh + kh - 1, ow + kw - 1, kh, kw, top=255.0)
    assert err2d(run2d(x, f, "AUTO"), x, f) <= TOL


@pytest.mark.parametrize("kh,kw", [(9, 13), (13, 13), (15, 15)])
@pytest.mark.parametrize("h", SEVERAL_CHUNKS)
def test_row_blocks_of_several_chunks(kh, kw, h):
    x, f = _case(h, 600, kh, kw)
    assert err2d(run2d(x, f, "AUTO"), x, f) <= TOL


@pytest.mark.parametrize("kh,kw", [(9, 13), (13, 13), (15, 15), (6, 14)])
@pytest.mark.parametrize("h", CUT_CHUNKS)
def test_blocks_that_end_inside_a_chunk(kh, kw, h):
    x, f = _case(h, 600, kh, kw, seed=1)
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


@pytest.mark.parametrize("kh,kw,h,w", [(13, 13, 60, 500), (15, 15, 60, 500), (9, 13, 300, 700), (11, 11, 1500, 1700)])
def test_numbers_of_two_and_three_parts_are_bit_exact(kh, kw, h, w):
    rng = np.random.default_rng(12)
    # 17 bits need two or three parts; 0 / 1 taps, at most 120 of them, keep every partial sum below 2^24
    x = rng.integers(-(1 << 17), 1 << 17, (h, w)).astype(np.float32)
    f = np.zeros(kh * kw, np.float32)
    f[rng.permutation(kh * kw)[:min(120, kh * kw - 3)]] = 1.0
    f = f.reshape(kh, kw)
    assert np.array_equal(run2d(x, f, "AUTO"), oracle.conv2d(x, f, ORACLE_THREADS).astype(np.float32))
    # a single tap of 1 picks an input out, all 24 bits of it
    x = _scaled((h, w), 1.0, seed=13)
    for p, q in [(0, 0), (kh - 1, kw - 1), (kh // 2, 3)]:
        f = np.zeros((kh, kw), np.float32)
        f[p, q] = 1.0
        assert np.array_equal(run2d(x, f, "AUTO"), x[p:p + h - kh + 1, q:q + w - kw + 1])


def _same_as_fbs(d, f):
    """AUTO against the FBS projection where both are finite, and the same infinities and NaN."""
    want, got = B.sys_conv2d(d, f, projection="FBS"), B.sys_conv2d(d, f)
    assert torch.equal(torch.isnan(want), torch.isnan(got)) and torch.equal(torch.isinf(want), torch.isinf(got))
    ok = torch.isfinite(want)
    scale = B.sys_conv2d(d.nan_to_num(0.0, 0.0, 0.0).abs(), np.abs(f), projection="FBS")
    assert ((want - got).abs()[ok] <= TOL * scale[ok]).all()


# Row blocks of 1 .. 56 chunks (32 with 4 x 4 offsets: the most that the rule takes; test_split_rules.py checks the heights), with one marked
# chunk early, late or in the last place, on either side of the 32nd and in the one that only finishes groups (row 16 n of n chunks), neighbouring ones, so many that a block is given up at once,
# half way or past the 32nd, and marks in each four rows of a chunk (53 rows apart), whose output rows overlap or do not.
MARKED_IMAGES = [(13, 13, 300, 500), (13, 13, 2900, 600), (10, 12, 30000, 600), (13, 13, 104000, 600), (15, 15, 171000, 600),
                 (13, 13, 63500, 741), (15, 15, 128000, 600), (15, 15, 143000, 600)]


@pytest.mark.parametrize("rows", [[3], [16 * 30], [16 * 62 + 5], [16 * 63], [40, 60, 900], list(range(500, 600, 16)), list(range(0, 1100, 16)),
                                  list(range(0, 1100, 96)), list(range(15, 1100, 112)), list(range(16, 32)), [7, 8], list(range(11, 1100, 53)),
                                  [2, 16 * 31 + 2], [16 * 32], [16 * 31 + 15, 16 * 32 + 9, 16 * 33], [16 * 47 + 3, 16 * 48 + 1], [16 * 55 + 15], [5, 16 * 56], [16 * 32 - 1, 16 * 56 + 14],
                                  list(range(16 * 33, 16 * 57, 16))])
@pytest.mark.parametrize("kh,kw,h,w", MARKED_IMAGES)
def test_marked_chunks_in_blocks_of_every_length(rows, kh, kw, h, w):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(kh)
    d = torch.rand((h, w), dtype=torch.float32, device="cuda", generator=gen)
    f = _case(kh, kw, kh, kw)[1]
    for i, r in enumerate(rows):
        if r < h:
            d[r, (97 * i) % w] = float("nan")
    if h > 20000:                                                          # a block far down, and the last rows of the image
        d[h - 1100:h - 1100 + len(rows) * 16:16, 5] = float("inf")
        d[h - 2, w - 1] = float("nan")
    _same_as_fbs(d, f)


def _scaled(shape, lo, seed):
    """Numbers of either sign with magnitudes in [lo, 2 lo)."""
    rng = np.random.default_rng(seed)
    return (np.ldexp(rng.uniform(1.0, 1.999, shape), int(np.log2(lo))) * rng.choice([-1.0, 1.0], shape)).astype(np.float32)


@pytest.mark.parametrize("kh,kw", [(13, 13), (15, 15)])
@pytest.mark.parametrize("tap,inputs", [
    # either side of the lower limit, 2^-100 over the smallest tap, and so far below it that the split alone would show
    (0.0, [-99, -100, -101, -130]), (-8.0, [-91, -92, -93, -122]), (-60.0, [-39, -40, -41, -58]),
    (5.0, [-102, -103, -104, -122]),                                       # large taps: 2^-103
    (0.0, [79, 80, 81]), (40.0, [79])])                                    # either side of the upper limit: sums just below 2^128
def test_either_side_of_the_limits(kh, kw, tap, inputs):
    f = _scaled((kh, kw), 2.0 ** tap, seed=8)
    f[1, 2] = 0.0
    for e in inputs:
        x = _scaled((150, 500), 2.0 ** e, seed=9)
        if e + tap > 100:
            x, f = (np.abs(x) / 2 + np.float32(2.0) ** (e - 1)).astype(np.float32), np.full((kh, kw), 2.0 ** tap, np.float32)
        assert err2d(run2d(x, f, "AUTO"), x, f) <= TOL, (tap, e)


def _us(fn, launches=6, best_of=5):
    fn()
    times = []
    for _ in range(best_of):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(launches):
            fn()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / launches)
    return min(times)


@pytest.mark.parametrize("kh,kw,vector", [(11, 11, "SBM"), (15, 15, "FBS")])
def test_no_input_makes_auto_much_slower_than_the_vector_kernels(kh, kw, vector):
    """Small values cost nothing; a NaN in every chunk costs what the vector kernels take and the chunks looked at before a
    block is given up (measured: 1.0 .. 1.35 times the vector kernel; the bound leaves room for another box's clocks)."""
    x, f = _case(4096, 4096, kh, kw, seed=10)
    d = dev(x)
    y = torch.empty(4097 - kh, 4097 - kw, dtype=torch.float32, device="cuda")
    plain, small, bound = (_us(lambda: B.sys_conv2d(d, f, y)), _us(lambda: B.sys_conv2d(d * 1e-15, f, y)),
                           _us(lambda: B.sys_conv2d(d, f, y, projection=vector)))
    scale = _us(lambda: d * 1e-15)
    assert small <= 1.5 * (plain + scale), f"{plain} {small}"
    d[5::16, 7::200] = float("nan")
    marked = _us(lambda: B.sys_conv2d(d, f, y))
    assert marked <= 2.0 * bound, f"a NaN per chunk: {marked:.1f} us, {vector} {bound:.1f} us"


def test_small_numbers_keep_their_precision():
    x, f = _case(80, 500, 13, 13, seed=4)
    for s in (1e-9, 1e-15, 1e-30, 1e-36, 1e15, 1e25):
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
