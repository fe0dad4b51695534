"""The threads per BFS of an untuned engine's fused launches, seen by their
slots (4,096 of one wave, 2,048 of 128 threads, 1,024 of 256): by the samples
and by the longest row of the pools' graphs, with the results of the plain
runs."""
import numpy as np
import pytest

from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def star(n):
    # undirected, a hub joined to every other node, and a ring
    v = np.arange(1, n)
    return inputs.from_edges(n, np.concatenate([np.zeros(n - 1, dtype=v.dtype), v]),
                             np.concatenate([v, np.roll(v, -1)]), directed=False)


@pytest.mark.parametrize("kinds,m,slots", [
    (("ba", "grid"), 20_000, 4096), (("ba", "grid"), 10_000, 2048), (("ba", "grid"), 1000, 1024),
    (("ba", "star"), 20_000, 2048), (("star",), 1000, 1000), (("grid", "grid"), 2500, 4096)])
def test_untuned_fused_launch(kinds, m, slots):
    make = {"ba": lambda: inputs.ba_graph(3000, 4, 7), "grid": lambda: inputs.grid_graph(32), "star": lambda: star(4000)}
    k, t, eps = 5, 8, 0.05
    ctx = binding.centra_create(0, 0)
    try:
        dgs = [binding.DeviceGraph(ctx, make[x]()) for x in kinds]
        eng = binding.Engine(ctx, 0, binding.CENTRA_ENGINE_NO_TUNE)
        try:
            say(f"fused launch over {kinds}, {m} samples each")
            qs = [eng.submit(eng.add_pool(dg.handle, 3, i, t, m, m), k, t, eps, 0.1) for i, dg in enumerate(dgs)]
            eng.run()
            assert eng.stats().sampler_launches == 1
            assert binding.centra_sampler_stats_get(ctx).slots == slots
            got = [eng.result(q) for q in qs]
        finally:
            eng.destroy()
        for i, (dg, g) in enumerate(zip(dgs, got)):
            rc, picks, res, _ = binding.centra_progressive(ctx, dg.handle, k, t, eps, 0.1, 3, i, m, m)
            assert rc == g[0] and np.array_equal(picks, g[1]) and res.coverage == g[2].coverage
            dg.release()
    finally:
        binding.centra_destroy(ctx)
