"""Histograms at the edges of the kernel's work split, against exact integer sums.

The expected values are the documented fixed-point sums themselves: every
value quantised to rint(v * 2^qexp) and added in int64, so the device's
histograms must equal them bit for bit.
"""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2211_12858_amd.driver import SplitSearch

pytestmark = pytest.mark.gpu


def exact_histograms(bins, GH, qexp, B, rows, off):
    """[node][feature][channel][bin] fp64, exact sums of the quantised values."""
    n_nodes, m, c = len(off) - 1, bins.shape[1], GH.shape[1]
    v = np.rint(np.ldexp(GH, qexp[None, :]).astype(np.float32)).astype(np.int64)
    H = np.zeros((n_nodes, m, c, B))
    for j in range(n_nodes):
        r = rows[off[j]:off[j + 1]]
        for f in range(m):
            for t in range(c):
                # integers below 2^53: the fp64 sums are exact
                H[j, f, t] = np.bincount(bins[r, f], weights=v[r, t].astype(np.float64), minlength=B)
    return np.ldexp(H, -qexp[None, None, :, None])


def case(n, m, B, k, seed):
    """Every fourth feature has a few levels only, one is constant; values reach the largest magnitude."""
    rng = np.random.default_rng(seed)
    bins = rng.integers(0, B, size=(n, m), dtype=np.uint8)
    for f in range(0, m, 4):
        bins[:, f] = rng.integers(0, 2 + f % 3, size=n, dtype=np.uint8) * ((B - 1) // 4)
    bins[:, m // 2] = B - 1
    GH = rng.uniform(-1, 1, size=(n, k + 1)).astype(np.float32)
    GH[:, 0] = np.float32(1.0) - np.float32(2.0 ** -24)  # quantises to 2^18 in every row
    GH[:, k] = 1.0
    return bins, GH, gu.qexp_rule(GH)


# rows: one step, one more and one less; several fold windows of 7680 rows in
# one row group (m = 300: few row groups); leftover features of every thin
# width (1, 2, 4, 8) and padded ones; bin counts off the staging's multiples
# of 32; one to three channel groups
@pytest.mark.parametrize("n,m,B,k", [(1, 1, 2, 1), (767, 16, 256, 5), (768, 17, 255, 5), (769, 18, 33, 4),
                                     (1537, 20, 34, 3), (5000, 24, 2, 2), (9000, 31, 64, 10), (3000, 49, 256, 16),
                                     (70_001, 300, 16, 5), (9000, 20, 256, 6), (9001, 33, 255, 7)])
def test_root_histograms_exact(n, m, B, k):
    bins, GH, qexp = case(n, m, B, k, seed=n + m)
    off = np.array([0, n], dtype=np.int32)
    H = gu.run_hist(bins, GH, qexp, B, None, off).cpu().numpy()
    assert np.array_equal(H, exact_histograms(bins, GH, qexp, B, np.arange(n), off))


@pytest.mark.parametrize("sizes,m,B,k", [([1, 0, 1, 1], 3, 256, 5), ([0, 0, 767, 0, 1, 768, 0], 17, 255, 5),
                                         ([2000, 1, 0, 3000, 769], 20, 33, 10), ([40_000, 5, 25_000], 260, 8, 5),
                                         ([7] * 40, 33, 64, 23), ([3000, 0, 1500], 18, 256, 7), ([900, 5], 40, 64, 6)])
def test_gathered_histograms_exact(sizes, m, B, k):
    n = sum(sizes) + 11
    bins, GH, qexp = case(n, m, B, k, seed=len(sizes) + m)
    rows = np.random.default_rng(1).permutation(n)[:sum(sizes)].astype(np.int32)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    H = gu.run_hist(bins, GH, qexp, B, rows, off).cpu().numpy()
    assert np.array_equal(H, exact_histograms(bins, GH, qexp, B, rows, off))


# The level loop's own reduction where a row group's sum of one bin leaves
# int32 (features of few levels, over 16384 rows per row group), with four
# threads per bin, one thread per bin and 12 channel pairs: the same trees as
# through the per-step calls, whose reduction the tests above check.
@pytest.mark.parametrize("n,m,k", [(200_000, 330, 5), (80_000, 1000, 5), (60_000, 300, 20)])
def test_tree_with_escaped_sums(n, m, k):
    bins, GH, qexp = case(n, m, 256, k, seed=k)
    rng = np.random.default_rng(7)
    G_T = rng.standard_normal((k, n)).astype(np.float32) + (bins[:, :k].T > 40)
    ss = SplitSearch(bins, 256, k, 2)
    ss.sketch("identity", torch.from_numpy(G_T.astype(np.float32)).to("cuda"), torch.ones(n, device="cuda"))
    ss.grow()
    a = ss.tree()
    ss.grow_levelwise()
    b = ss.tree()
    for l in range(2):
        for key in ("feature", "bin", "score"):
            assert np.array_equal(a[key][l], b[key][l]), (l, key)
    assert np.array_equal(a["row_idx"], b["row_idx"])
