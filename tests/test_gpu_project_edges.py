"""The dense projection's two block forms (2048 and 512 rows each) at the edges of their use, within the dot-product
error bound."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


def check_projection(n, d, k, rows=slice(None)):
    rng = np.random.default_rng(n + d + k)
    G_T = rng.random((d, n), dtype=np.float32) - np.float32(0.5)
    Pi = (rng.standard_normal((d, k)) / np.sqrt(k)).astype(np.float32)
    h = rng.uniform(0.5, 1.0, n).astype(np.float32)
    GH, _, _, _, qexp, pad = gu.run_sketch("random_projection", G_T, h, k, Pi=Pi)
    G64, Pi64 = G_T[:, rows].T.astype(np.float64), Pi.astype(np.float64)
    want = G64 @ Pi64
    u = 2.0 ** -24
    gamma = d * u / (1 - d * u)
    err = np.abs(GH[rows, :k].astype(np.float64) - want)
    assert np.all(err <= gamma * (np.abs(G64) @ np.abs(Pi64)) + u * np.abs(want) + 1e-30)
    assert np.array_equal(GH[:, k], h)
    assert np.array_equal(qexp, gu.qexp_rule(GH))
    assert not pad.any()


# 230 blocks of 2048 rows (the fewest that take them), with a ragged last one
# whose last lane holds one row; a full last block; one block more than 256
# (small blocks again); every register form (8 to 24 columns) and a width past
# it; in one round 100 columns of G are the fewest that take them up to k = 12 and
# 50 up to k = 23, and one less; at k = 24 any number
@pytest.mark.parametrize("n,d,k", [(229 * 2048 + 1, 100, 8), (230 * 2048, 100, 12), (230 * 2048 + 127, 51, 13),
                                   (256 * 2048, 50, 20), (256 * 2048 - 1, 3, 24), (256 * 2048 + 1, 100, 20),
                                   (230 * 2048, 3, 25), (230 * 2048, 99, 8), (230 * 2048, 49, 16),
                                   (230 * 2048 + 1, 50, 21)])
def test_large_blocks(n, d, k):
    check_projection(n, d, k)


# Two rounds of large blocks (460 is the fewest that fill 0.9 of 512): 200 columns
# of G are the fewest that take them there, and one less; past 256 columns two staged
# blocks of Pi.
@pytest.mark.parametrize("d", [199, 200, 257])
def test_large_blocks_two_rounds(d):
    n = 460 * 2048 - 1
    rows = np.r_[0:4096, n // 2:n // 2 + 4096, n - 4096:n]
    check_projection(n, d, 9, rows)


# Small blocks: every number of column groups (k = 33 is a second pass of one),
# rows in pairs and in runs of 64, one row to one more than a block, columns of
# G around a batch of 16 and a staged block of 256.
@pytest.mark.parametrize("n,d", [(1, 17), (127, 15), (512, 256), (513, 257), (1100, 16)])
@pytest.mark.parametrize("k", [8, 12, 16, 20, 24, 28, 32, 33])
def test_small_blocks(n, d, k):
    check_projection(n, d, k)
