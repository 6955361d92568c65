"""The one-block partition of small levels at the edges of its use: rows around its blocks of 1024 and its
limits (4096 and 10240 rows), nodes around its limit of 32 and, as a call of its own, 16 x 10240 rows x nodes, as
inputs and inside whole trees (which have the limit of 32 nodes only)."""
import numpy as np
import pytest
import torch

from paper_2211_12858_amd.driver import SplitSearch
from test_gpu_calls import test_partition_bit_exact as partition_bit_exact
from workloads import small_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_nodes", [(1, 1), (63, 2), (1023, 31), (1024, 32), (1025, 33), (4096, 32), (4097, 3),
                                       (10240, 16), (10240, 17), (5120, 32), (5121, 32), (10240, 32), (10240, 33),
                                       (10241, 16)])
def test_partition(n, n_nodes):
    partition_bit_exact(n, 6, n_nodes, seed=n + n_nodes)


@pytest.mark.parametrize("n", [700, 4097, 10240, 10241])
def test_tree(n):
    # the level loop picks the splits inside the partition (depth 7: levels of
    # up to 64 nodes, on both sides of the limit); the per-step calls do not, and
    # take two launches from 17 nodes on at 10,240 rows
    case = small_case(n, 70, 64, 4, seed=n)
    ss = SplitSearch(case.bins, 64, 4, 7)
    ss.sketch("identity", torch.from_numpy(case.G_T).to("cuda"), torch.from_numpy(case.h).to("cuda"))
    ss.grow()
    a = ss.tree()
    ss.grow_levelwise()
    b = ss.tree()
    for key in ("feature", "bin", "score"):
        for x, y in zip(a[key], b[key]):
            assert np.array_equal(x, y), key
    assert np.array_equal(a["row_idx"], b["row_idx"]) and np.array_equal(a["leaf_off"], b["leaf_off"])
