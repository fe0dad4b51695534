"""kappa-path walks against the oracle on either side of the walk sizes the
kernel is built for (4, 8 and 16 nodes), on graphs whose rows are one entry,
a power of two around which the search's halves change, and used up by the
walk."""
import numpy as np
import pytest

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say

pytestmark = pytest.mark.gpu


def complete(n):
    a, b = np.triu_indices(n, 1)
    return inputs.from_edges(n, a, b, directed=False)


GRAPHS = {
    "pair": lambda: complete(2),
    "k5": lambda: complete(5),
    "k9": lambda: complete(9),
    "k18": lambda: complete(18),
    "ring_of_hubs": lambda: inputs.from_edges(
        200, np.concatenate([np.arange(40)] + [np.full(127 + d, d) for d in range(3)]),
        np.concatenate([(np.arange(40) + 1) % 40] + [np.arange(60, 187 + d) for d in range(3)]), directed=False),
    "dag": lambda: inputs.from_edges(12, *np.triu_indices(12, 1), directed=True),
}


@pytest.mark.parametrize("kappa", [4, 5, 7, 8, 9, 16])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_walk_sizes(name, kappa):
    g = GRAPHS[name]()
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"kpaths {name} kappa {kappa}")
            off, nodes = binding.sample_kpaths(ctx, dg, kappa, 5, 1, 7, 3000)
            want_off, want_nodes = oracle.sample_kpaths(g, kappa, 5, 1, 7, 3000)
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
