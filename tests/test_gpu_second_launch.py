"""centra_sample_paths on graphs where many searches outgrow the launch's scan
budget: they are drawn by a second launch, not one after another by the
device-wide BFS, with the same hyperedges; and what a second launch defers
still ends on the device-wide BFS."""
import numpy as np
import pytest
import torch

from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, oracle_paths, say

pytestmark = pytest.mark.gpu


def long_in_rows(n, d, seed):
    # directed, d out-arcs per node, targets skewed: searches reach most nodes
    rng = np.random.default_rng(seed)
    src = np.repeat(np.arange(n), d)
    dst = rng.permutation(n)[(rng.random(n * d) ** 3 * n).astype(np.int64)]
    keep = src != dst
    return inputs.from_edges(n, src[keep], dst[keep], directed=True)


def draw(ctx, dg, count):
    binding.centra_sampler_stats_get(ctx, reset=True)
    off, nodes, st, dist = binding.sample_paths(ctx, dg, 5, 0, 0, count, with_st=True)
    return off_np(off), nodes_np(nodes), nodes_np(st), nodes_np(dist), binding.centra_sampler_stats_get(ctx)


@pytest.mark.parametrize("wide_nodes", [None, "300"])
def test_many_deferred(wide_nodes, monkeypatch):
    g, count = long_in_rows(100_000, 8, 1), 6000
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            monkeypatch.setenv("CENTRA_WIDE", "0")
            want = draw(ctx, dg, count)
            monkeypatch.delenv("CENTRA_WIDE")
            if wide_nodes:
                monkeypatch.setenv("CENTRA_WIDE_NODES", wide_nodes)
            got = [draw(ctx, dg, count) for _ in range(2)]
            say(f"{count} samples, wide levels from {wide_nodes}: device-wide {[x[4].wide for x in got]}, "
                f"arcs {[x[4].arcs for x in got]} ({want[4].arcs} without)")
            for x in got:
                assert all(np.array_equal(a, b) for a, b in zip(x[:4], want[:4]))
                assert x[4].samples == count and x[4].launches == 1
                # searches were left and drawn again, at most a few of them device-wide
                assert x[4].arcs > want[4].arcs if wide_nodes is None else x[4].wide > 8
                assert wide_nodes is not None or x[4].wide <= 8
            for i, w in zip(range(0, count, 97), oracle_paths(g, 5, 0, range(0, count, 97), dg.info()[1])):
                assert np.array_equal(want[1][int(want[0][i]):int(want[0][i + 1])], w[0])
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
