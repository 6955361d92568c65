"""The gradient passes at the edges of their tiles.

First the one-pass update + derivatives of the sigmoid loss, against the two calls it stands for:

Column chunks of 16 (d around multiples of 16), row tiles of 256 (ragged and
full, one and several per block, more tiles than norm slots) and leaf counts up
to the 256 that one pass takes (and one more, which takes the two calls): bit
for bit, norms included.
"""
import numpy as np
import pytest

from test_gpu_boost import check_gradients
from test_gpu_boost import test_update_and_gradients_bit_exact as update_and_gradients_bit_exact
from workloads import scores_and_targets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n_leaves,n", [(1, 1, 1), (15, 2, 255), (16, 128, 256), (17, 256, 257), (33, 255, 770 * 256),
                                          (48, 31, 1536 * 256 + 1), (203, 128, 3001), (20, 257, 2000)])
def test_sigmoid_update_and_gradients(d, n_leaves, n):
    update_and_gradients_bit_exact("sigmoid", d, n_leaves, n)


# The register softmax of wide rows: columns around multiples of 32 (a wave's
# columns) and of 64 (past 512, where a wave's lanes are two halves of columns),
# its ends 105 and 1024 and the first width past them; row tiles of 64 and 32,
# ragged, one block to several tiles per block; against the fp64 oracle.
@pytest.mark.parametrize("d,n", [(105, 1), (128, 63), (129, 64), (160, 65), (200, 70_003), (511, 300), (512, 257),
                                 (513, 31), (544, 32), (577, 33), (640, 9001), (1000, 515), (1024, 257), (1025, 100)])
def test_wide_softmax_gradients(d, n):
    F_T, y = scores_and_targets(n, d, "softmax", seed=d + n, scale=2.0)
    G1, H1, hr1, n1 = check_gradients("softmax", F_T, y)
    G2, H2, hr2, n2 = check_gradients("softmax", F_T, y)
    assert np.array_equal(G1, G2) and np.array_equal(H1, H2) and np.array_equal(hr1, hr2) and np.array_equal(n1, n2)


# The two-pass softmax past 1024 columns: a full tile of 256 rows alone, with a
# ragged one, and several, with one ragged last chunk of columns.
@pytest.mark.parametrize("d,n", [(1025, 256), (1025, 257), (1041, 770)])
def test_two_pass_softmax_gradients(d, n):
    F_T, y = scores_and_targets(n, d, "softmax", seed=d + n, scale=2.0)
    check_gradients("softmax", F_T, y)


# A leading dimension of 2^24 takes narrower rows to the two-pass kernel too
# (below it, the wide kernel): more tiles than the 1536 norm slots, so slots take two.
def test_two_pass_softmax_by_leading_dimension():
    F_T, y = scores_and_targets(1536 * 256 + 300, 106, "softmax", seed=5, scale=2.0)
    check_gradients("softmax", F_T, y, ld_f=1 << 24)
