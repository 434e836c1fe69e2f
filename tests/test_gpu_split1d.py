"""The 1-D matrix-core kernel behind AUTO (28 taps and more): edges of its tiles (256 outputs) and runs of tiles, both instruction
counts, and the inputs that its three-part split does not carry.

Tolerance: the split is exact, six of nine products are kept and accumulated in fp32; 64 taps round at most 64 times in any
order, 64 * 2^-24 = 3.8e-6 of the scale, inside the parity metric's 1e-5.  Integers whose products and sums stay below 2^24 need
one part each and come out bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import TOL, dev, err1d, run1d
from paper_2010_15884_amd import binding as B

pytestmark = pytest.mark.gpu

TAPS = [28, 33, 49, 50, 64]                # 49 / 50: the step from two to three instructions


def _case(n, k, seed=0):
    rng = np.random.default_rng(1000 * k + n + seed)
    return rng.uniform(-1, 1, n).astype(np.float32), rng.uniform(-1, 1, k).astype(np.float32)


@pytest.mark.parametrize("k", TAPS)
def test_auto_runs_the_split_kernel(k):
    """FBS, BFS and SBM add an output's taps in an order of their own; the split's sums round elsewhere.  27 taps stay with FBS."""
    x, w = _case(5000, k)
    auto = B.sys_conv1d(dev(x), w)
    for proj in ("FBS", "SBM", "BFS"):
        assert (auto != B.sys_conv1d(dev(x), w, projection=proj)).float().mean() > 0.2, proj
    assert torch.equal(B.sys_conv1d(dev(x), w[:27]), B.sys_conv1d(dev(x), w[:27], projection="FBS"))


@pytest.mark.parametrize("k", TAPS)
# one output, one quad, a tile, a workgroup of one-tile runs, and more
@pytest.mark.parametrize("m", [1, 3, 4, 15, 17, 255, 256, 257, 511, 512, 1023, 1025, 1280, 70001])
def test_edges_of_tiles(k, m):
    x, w = _case(m + k - 1, k)
    assert err1d(run1d(x, w, "AUTO"), x, w) <= TOL


# runs of 2, 3, 5 and 9 tiles, the last one cut; past 33.5 M a second round (runs of 8 up to 49 taps), past 37.7 M the non-temporal loads
@pytest.mark.parametrize("n,k", [(1_100_003, 50), (2_900_001, 33), (4_300_007, 64), (9_000_001, 49), (34_000_003, 28), (38_000_001, 50),
                                 (38_000_001, 49)])
def test_runs_of_several_tiles(n, k):
    x, w = _case(n, k)
    assert err1d(run1d(x, w, "AUTO"), x, w) <= TOL


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("n,k", [(9001, 50), (300, 33)])
def test_integers_exact_unaligned_and_nothing_written_outside(n, k, off):
    rng = np.random.default_rng(7)
    x, w = rng.integers(-100, 100, n).astype(np.float32), rng.integers(-9, 9, k).astype(np.float32)
    xbuf = torch.full((n + 8,), float("nan"), dtype=torch.float32, device="cuda")
    xbuf[off:off + n] = dev(x)
    ybuf = torch.full((n + 64,), float("nan"), dtype=torch.float32, device="cuda")
    m = n - k + 1
    B.sys_conv1d(xbuf[off:off + n], w, ybuf[32 + off:32 + off + m])
    out = ybuf.cpu().numpy()
    assert np.isnan(out[:32 + off]).all() and np.isnan(out[32 + off + m:]).all()
    assert np.array_equal(out[32 + off:32 + off + m].astype(np.float64), oracle.conv1d(x, w))


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 2.0 ** 90, 2.0 ** -110, 1e-41])
@pytest.mark.parametrize("n,k", [(300, 28), (1500, 50), (1_300_003, 64)])      # one tile, one-tile runs, runs of two
def test_values_the_split_does_not_carry(value, n, k):
    """At the signal's ends, around a tile's and a run's edge, alone and in a stretch: bit for bit what plain sums give on the outputs that
    see one (BFS, the same order), within the tolerance elsewhere, and no other output is touched by a NaN."""
    x, w = _case(n, k, 3)
    spots = [p for p in (0, 254, 255, 256, 511, 513, 700, n // 2, n - 1) if p < n]
    x[spots] = value
    if n > 3000:
        x[2000:2900] = value
    y, plain = run1d(x, w, "AUTO"), run1d(x, w, "BFS")
    seen = np.convolve(x == np.float32(value) if value == value else np.isnan(x), np.ones(k), "valid") > 0.5
    assert np.array_equal(y[seen], plain[seen], equal_nan=True)
    if (~seen).any():
        clean = np.where(np.isfinite(x), x, 0)
        ref, scale = oracle.conv1d(clean, w), oracle.absdot1d(clean, w)
        assert oracle.max_rel_err(y[~seen], ref[~seen], scale[~seen]) <= TOL


@pytest.mark.parametrize("tap", [2.0 ** -61, 2.0 ** 41])
def test_taps_the_split_does_not_carry(tap):
    x, w = _case(3000, 40)
    w[7] = tap
    assert torch.equal(B.sys_conv1d(dev(x), w), B.sys_conv1d(dev(x), w, projection="BFS"))
