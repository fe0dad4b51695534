"""Greedy cover on many short hyperedges over few nodes: samples on either side
of their share of one workgroup's entries per round, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say
from tests.test_gpu_greedy_batch_rule import cover

pytestmark = pytest.mark.gpu


# samples of one node: with two more entries for each past 65,536, at k * 12,288 and past it
@pytest.mark.parametrize("m,k", [(65_536, 6), (65_537, 5), (88_746, 11), (88_747, 11), (92_842, 12), (92_843, 12)])
@pytest.mark.parametrize("n", [7, 500])
def test_one_node_each(n, m, k):
    rng = np.random.default_rng(m)
    off = np.arange(m + 1, dtype=np.uint64)
    nodes = np.minimum((n * rng.random(m) ** 2), n - 1).astype(np.uint32)
    say(f"greedy n {n} m {m} k {k}")
    picks, cov = cover(n, off, nodes, k)
    want_picks, want_cov = oracle.greedy_cover(n, off, nodes, k)
    assert picks == list(want_picks)
    assert cov == list(want_cov)
