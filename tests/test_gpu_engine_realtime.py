"""Realtime engine runs of few queries: a query alone, or with queries of other
pools about to arrive, goes from level to level without a pause; one of its
own pool that is due within 3 ms joins it."""
import pytest

from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

LEVELS = 8   # 500, 1000, ..., 64000


def serve(ctx, dgs, queries):
    """Runs (pool, arrival) queries in real time; their infos and the stats."""
    eng = binding.Engine(ctx, 0, binding.CENTRA_ENGINE_NO_TUNE)
    try:
        pids = [eng.add_pool(dg.handle, 5, i, 8, 500, 64_000) for i, dg in enumerate(dgs)]
        qids = [eng.submit(pids[p], 5, 8, 0.001, 0.1, a) for p, a in queries]
        eng.run(realtime=True)
        got = [eng.result(q) for q in qids]
        assert all(g[2].iterations == LEVELS for g in got)
        return [g[3] for g in got], eng.stats()
    finally:
        eng.destroy()


def test_no_pause_without_a_neighbour():
    g = inputs.ba_graph(300, 3, 4)
    ctx = binding.centra_create(0, 0)
    dgs = [binding.DeviceGraph(ctx, g), binding.DeviceGraph(ctx, g)]
    try:
        for queries in ([(0, 0.0)], [(0, 0.0), (1, 0.5)], [(0, 0.0), (0, 0.5)]):
            serve(ctx, dgs, queries)   # workspaces, captured graphs
            took = min((i[0].finished_s - i[0].admitted_s) * 1e3 for i in (serve(ctx, dgs, queries)[0] for _ in range(5)))
            say(f"{len(queries)} queries {queries}: the first takes {took:.2f} ms for {LEVELS} levels")
            # a pause to 1.5 ms after each level but the last took 10.5 ms at least
            assert took < (LEVELS - 1) * 1.5
    finally:
        for dg in dgs:
            dg.release()
        binding.centra_destroy(ctx)


def test_a_neighbour_of_the_pool_is_joined():
    # the second query is due well before the first could draw its levels and
    # 3 ms after it at most: they are active together
    g = inputs.ba_graph(300, 3, 4)
    ctx = binding.centra_create(0, 0)
    dgs = [binding.DeviceGraph(ctx, g), binding.DeviceGraph(ctx, g)]
    try:
        serve(ctx, dgs, [(0, 0.0)])
        infos, st = serve(ctx, dgs, [(0, 0.0), (0, 0.0025)])
        assert st.peak_active == 2 and infos[1].admitted_s >= 0.0025 - 1e-9
        assert infos[0].finished_s > infos[1].admitted_s
    finally:
        for dg in dgs:
            dg.release()
        binding.centra_destroy(ctx)
