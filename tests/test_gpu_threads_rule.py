"""How many threads the path sampler gives a BFS, seen by the slots of a launch
of more samples than it holds at once (4,096 of one wave, 2,048 of 128
threads, 1,024 of 256): by the number of samples, by the shape of the graph
and by the memory for slots; and parity with the oracle on each side."""
import numpy as np
import pytest

from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, oracle_paths, say

pytestmark = pytest.mark.gpu


def ring(n, strides, directed):
    v = np.arange(n)
    return inputs.from_edges(n, np.tile(v, len(strides)), np.concatenate([(v + s) % n for s in strides]),
                             directed=directed)


def hub_in(n):
    # directed, at most 4 out-arcs per node, one in-row of n / 4 entries
    v = np.arange(n)
    src = np.concatenate([v, v, v[::4]])
    dst = np.concatenate([(v + 1) % n, (v + 61) % n, np.zeros(len(v[::4]), dtype=v.dtype)])
    keep = src != dst
    return inputs.from_edges(n, src[keep], dst[keep], directed=True)


GRAPHS = {"grid": lambda: inputs.grid_graph(64), "grid200": lambda: inputs.grid_graph(200), "hub_in": lambda: hub_in(4096),
          "ring16": lambda: ring(4096, [1, 9, 77, 200, 511, 900, 1500, 2000], False),
          "ba": lambda: inputs.ba_graph(3000, 3, 2), "tiny": lambda: inputs.ba_graph(300, 5, 1)}


@pytest.mark.parametrize("kind,count,budget_mb,slots", [
    ("grid", 5000, 0, 4096), ("grid", 4095, 0, 2048), ("grid", 2047, 0, 1024),
    ("grid200", 5000, 0, 2048), ("hub_in", 5000, 0, 2048), ("ring16", 5000, 0, 2048),
    ("ba", 32_767, 0, 2048), ("ba", 32_768, 0, 4096), ("ba", 2048, 0, 2048), ("ba", 2047, 0, 1024),
    ("tiny", 40_000, 1000, 1024), ("tiny", 40_000, 2000, 2048), ("tiny", 40_000, 4000, 2048),
    ("tiny", 40_000, 40_000, 4096)])
def test_threads_per_bfs(kind, count, budget_mb, slots):
    g = GRAPHS[kind]()
    ctx = binding.centra_create(0, budget_mb << 20)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"{kind}: {count} samples, budget {budget_mb} MB")
            off, nodes = binding.sample_paths(ctx, dg, 7, 1, 0, count)
            assert binding.centra_sampler_stats_get(ctx).slots == slots
            off, nodes = off_np(off), nodes_np(nodes)
            some = range(0, count, 211)
            for i, w in zip(some, oracle_paths(g, 7, 1, some, dg.info()[1])):
                assert np.array_equal(nodes[int(off[i]):int(off[i + 1])], w[0])
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
