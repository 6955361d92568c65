"""The one-pass update + derivatives of the sigmoid loss at its edges, against the two calls it stands for.

Column chunks of 16 (d around multiples of 16), row tiles of 256 (ragged and
full, one and several per block, more tiles than norm slots) and leaf counts up
to the 256 that one pass takes (and one more, which takes the two calls): bit
for bit, norms included.
"""
import pytest

from test_gpu_boost import test_update_and_gradients_bit_exact as update_and_gradients_bit_exact

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n_leaves,n", [(1, 1, 1), (15, 2, 255), (16, 128, 256), (17, 256, 257), (33, 255, 770 * 256),
                                          (48, 31, 1536 * 256 + 1), (203, 128, 3001), (20, 257, 2000)])
def test_sigmoid_update_and_gradients(d, n_leaves, n):
    update_and_gradients_bit_exact("sigmoid", d, n_leaves, n)
