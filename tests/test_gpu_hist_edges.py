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


# rows: one step, one more and one less; several steps of a row group (m = 300: few
# row groups); leftover features of every thin width (1, 2, 4, 8) and padded ones; bin
# counts off the staging's multiples of 32; one to three channel groups
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


# ---------------------------------------------------------------- long row groups
WINDOW = 7680          # rows between two folds of a row group's LDS sums
TOP = np.float32(1.0) - np.float32(2.0 ** -24)  # quantises to 2^18


def row_groups(m, c):
    """Row groups of a full slice on a large level, m a multiple of 16 (the kernel's documented split of 256 CUs)."""
    assert m % 16 == 0
    units = m // 16 * -(-c // 6)  # (slice, channel group) workgroups of a row group
    q = max(256 // units, 1)
    best = -(-q * units // 256) / q
    for more in range(q + 1, 9):
        cost = -(-more * units // 256) / more
        if cost < 0.95 * best:
            q, best = more, cost
    return q


def exact_sums(bins, v, B, rows):
    """[feature][channel][bin] int64 sums of the quantised values v (n, c) over the given rows."""
    b = torch.from_numpy(bins[rows]).to("cuda").long()
    v = torch.from_numpy(v[rows]).to("cuda")
    m, c = b.shape[1], v.shape[1]
    at = (torch.arange(m, device="cuda") * B + b).reshape(-1)
    out = torch.zeros((c, m * B), dtype=torch.int64, device="cuda")
    for t in range(c):
        out[t].index_add_(0, at, v[:, t:t + 1].expand(-1, m).reshape(-1))
    return out.view(c, m, B).permute(1, 0, 2).cpu().numpy()


# Row groups of more than two fold windows with a ragged last one, every number of
# channels a workgroup takes (k = 7: two groups of four), and 256 bins with a
# single row group.  Channels of +2^18 and of -2^18 in every row, in both halves of
# a pair: a constant feature's cell changes by 0.94 of 2^31 in a window, and its
# partial sum leaves int32.
@pytest.mark.parametrize("gathered", [False, True])
@pytest.mark.parametrize("n,m,B,k", [(40_001, 2000, 16, 1), (40_001, 2000, 8, 2), (40_001, 2000, 16, 3),
                                     (40_001, 2000, 8, 4), (40_001, 2000, 16, 5), (40_001, 1008, 8, 7),
                                     (16_001, 4096, 256, 5)])
def test_row_groups_of_several_windows(n, m, B, k, gathered):
    q = row_groups(m, k + 1)
    assert n // q > 2 * WINDOW and n // q % WINDOW
    rng = np.random.default_rng(n + m + k)
    bins = rng.integers(0, B, size=(n, m), dtype=np.uint8)
    bins[:, 0] = 0
    bins[:, m // 2] = B - 1
    bins[:, m - 1] = rng.integers(0, 2, size=n)
    GH = rng.uniform(-1, 1, size=(n, k + 1)).astype(np.float32)
    for t in range(min(4, k + 1)):
        GH[:, t] = TOP if t < 2 else -TOP
    qexp = gu.qexp_rule(GH)
    v = np.rint(np.ldexp(GH, qexp[None, :]).astype(np.float32)).astype(np.int64)
    if gathered:
        rows = rng.permutation(n).astype(np.int32)
        off = np.array([0, 3 * n // 4, 3 * n // 4, n], dtype=np.int32)
    else:
        rows, off = None, np.array([0, n], dtype=np.int32)
    H = gu.run_hist(bins, GH, qexp, B, rows, off).cpu().numpy()
    for j in range(len(off) - 1):
        at = slice(off[j], off[j + 1]) if rows is None else rows[off[j]:off[j + 1]]
        want = exact_sums(bins, v, B, at)
        assert np.abs(want).max() >= (1 << 18) * int(off[j + 1] - off[j])
        assert np.array_equal(H[j], np.ldexp(want.astype(np.float64), -qexp[None, :, None])), j


# The level loop's own reduction where a row group's sum of one bin leaves
# int32, with four threads per bin, one thread per bin and 12 channel pairs.  The
# hessians quantise to 2^18, so a feature of two levels escapes above 8192 rows of a
# level in a row group, and the gradients follow one such feature, whose sums
# escape too: the tree splits on it, with the score of the exact integer sums, and
# agrees with the per-step calls, whose reduction the tests above check.
@pytest.mark.parametrize("n,m,k", [(240_000, 320, 5), (80_000, 992, 5), (60_000, 304, 20)])
def test_tree_with_escaped_sums(n, m, k):
    assert n // row_groups(m, k + 1) > 2.2 * 8192
    B, lam, split = 256, 1.0, 8
    rng = np.random.default_rng(n + k)
    bins = rng.integers(0, B, size=(n, m), dtype=np.uint8)
    for f in range(0, m, 4):
        bins[:, f] = rng.integers(0, 2, size=n, dtype=np.uint8) * 63
    bins[:, m // 2 + 1] = B - 1
    side = np.where(bins[:, split] > 0, np.float32(0.95), np.float32(-0.95))
    G_T = (rng.uniform(-0.04, 0.04, size=(k, n)).astype(np.float32) + side).astype(np.float32)
    GH = np.concatenate([G_T.T, np.full((n, 1), TOP, dtype=np.float32)], axis=1)
    ss = SplitSearch(bins, B, k, 2, lam)
    ss.sketch("identity", torch.from_numpy(G_T).to("cuda"), torch.full((n,), float(TOP), device="cuda"))
    ss.grow()
    a = ss.tree()
    ss.grow_levelwise()
    b = ss.tree()
    for l in range(2):
        for key in ("feature", "bin", "score"):
            assert np.array_equal(a[key][l], b[key][l]), (l, key)
    assert np.array_equal(a["row_idx"], b["row_idx"])

    qexp = gu.qexp_rule(GH)
    v = np.rint(np.ldexp(GH, qexp[None, :]).astype(np.float32)).astype(np.int64)
    H = np.ldexp(exact_sums(bins, v, B, np.arange(n)).astype(np.float64), -qexp[None, :, None])
    left = np.cumsum(H, axis=2)[:, :, :-1]
    right = H.sum(axis=2, keepdims=True) - left
    ok = (left[:, k] > 0) & (right[:, k] > 0)
    S = (left[:, :k] ** 2).sum(axis=1) / (left[:, k] + lam) + (right[:, :k] ** 2).sum(axis=1) / (right[:, k] + lam)
    S[~ok] = -np.inf
    f, t = np.unravel_index(np.argmax(S), S.shape)
    assert f == split and (a["feature"][0][0], a["bin"][0][0]) == (f, t)
    # (at most 24 channels' squares, each with a few roundings)
    assert abs(a["score"][0][0] - S[f, t]) <= 64 * 2.0 ** -53 * S[f, t]
