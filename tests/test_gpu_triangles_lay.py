"""Triangles laid out in rank order, every rank read by some sample: groups of
arcs without a triangle, with one, with more than a workgroup's threads, and a
last group that is not full; with and without a budget (under which the rest
of the index is given back)."""
import itertools

import numpy as np
import pytest

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say

pytestmark = pytest.mark.gpu


def path_then_clique(n, k):
    # a path of n nodes (no triangle), its end in a clique of k nodes
    e = [(i, i + 1) for i in range(n - 1)]
    e += [(n - 1 + i, n - 1 + j) for i, j in itertools.combinations(range(k), 2)]
    return inputs.from_edges(n - 1 + k, *zip(*e), directed=False)


def wheel(n):
    e = [(0, i) for i in range(1, n)] + [(i, i + 1) for i in range(1, n - 1)] + [(1, n - 1)]
    return inputs.from_edges(n, *zip(*e), directed=False)


GRAPHS = {"k90": lambda: inputs.from_edges(90, *zip(*itertools.combinations(range(90), 2)), directed=False),
          "path-k30": lambda: path_then_clique(700, 30), "wheel": lambda: wheel(2001),
          "one": lambda: path_then_clique(100, 3), "ba": lambda: inputs.ba_graph(3000, 6, 3)}


@pytest.mark.parametrize("budget_mb", [0, 1000])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_every_rank(name, budget_mb):
    g = GRAPHS[name]()
    T = len(oracle.triangles(g))
    count = min(12 * T, 400_000)
    ctx = binding.centra_create(0, budget_mb << 20)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"triangles laid out: {name}, T {T}, budget {budget_mb} MB, {count} samples")
            assert binding.centra_triangle_count(ctx, dg.handle) == T
            off, nodes = binding.sample_triangles(ctx, dg, 2, 1, 0, count)
            want_off, want_nodes = oracle.sample_triangles(g, 2, 1, 0, count)
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
