"""kappa-path walks of 9 to 16 nodes against the oracle, on rows of hundreds of
entries and on rows that the walk uses up."""
import numpy as np
import pytest

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say

pytestmark = pytest.mark.gpu

GRAPHS = {"ba": lambda: inputs.ba_graph(3000, 5, 4), "rmat": lambda: inputs.rmat_graph(10, 8, seed=5),
          "grid": lambda: inputs.grid_graph(9),
          "k11": lambda: inputs.from_edges(11, *np.triu_indices(11, 1), directed=False)}


@pytest.mark.parametrize("kappa", range(9, 17))
@pytest.mark.parametrize("name", list(GRAPHS))
def test_long_walks(name, kappa):
    g = GRAPHS[name]()
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"kpaths {name} kappa {kappa}: 5000 walks")
            off, nodes = binding.sample_kpaths(ctx, dg, kappa, 5, 1, 3, 5000)
            want_off, want_nodes = oracle.sample_kpaths(g, kappa, 5, 1, 3, 5000)
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
