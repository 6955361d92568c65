"""The dense projection's large blocks (2048 rows each) at the edges of their use, within the dot-product error bound."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


# 230 blocks of 2048 rows (the fewest that take them), with a ragged last one
# whose last lane holds one row; a full last block; one block more than 256
# (small blocks again); every register form (8 to 24 columns) and a width past it
@pytest.mark.parametrize("n,k", [(229 * 2048 + 1, 8), (230 * 2048, 12), (230 * 2048 + 127, 13), (256 * 2048, 20),
                                 (256 * 2048 - 1, 24), (256 * 2048 + 1, 20), (230 * 2048, 25)])
def test_large_blocks(n, k):
    d = 3
    rng = np.random.default_rng(k)
    G_T = rng.standard_normal((d, n)).astype(np.float32)
    Pi = (rng.standard_normal((d, k)) / np.sqrt(k)).astype(np.float32)
    h = rng.uniform(0.5, 1.0, n).astype(np.float32)
    GH, _, _, _, qexp, pad = gu.run_sketch("random_projection", G_T, h, k, Pi=Pi)
    G64, Pi64 = G_T.T.astype(np.float64), Pi.astype(np.float64)
    want = G64 @ Pi64
    u = 2.0 ** -24
    gamma = d * u / (1 - d * u)
    err = np.abs(GH[:, :k].astype(np.float64) - want)
    assert np.all(err <= gamma * (np.abs(G64) @ np.abs(Pi64)) + u * np.abs(want) + 1e-30)
    assert np.array_equal(GH[:, k], h)
    assert np.array_equal(qexp, gu.qexp_rule(GH))
    assert not pad.any()
