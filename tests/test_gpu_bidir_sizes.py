"""GPU parity of the bidirectional sampler where its paths part: levels around
one wave's nodes and the arcs of the small expansion, meeting sets around and
past what the LDS table holds, count shifts (which rule the look-ahead out),
for every thread count per search."""
import numpy as np
import pytest

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say
from tests.test_gpu_bidir import budgets

pytestmark = pytest.mark.gpu


def layers(widths, directed):
    # a chain of layers of the given widths, neighbouring layers fully joined
    ids, first = [], 0
    for w in widths:
        ids.append(np.arange(first, first + w))
        first += w
    src = np.concatenate([np.repeat(a, len(b)) for a, b in zip(ids, ids[1:])])
    dst = np.concatenate([np.tile(b, len(a)) for a, b in zip(ids, ids[1:])])
    if directed:   # and back, so that pairs are reachable both ways
        src, dst = np.concatenate([src, [first - 1]]), np.concatenate([dst, [0]])
    return inputs.from_edges(first, src, dst, directed=directed)


WIDTHS = {
    "waves": (1, 63, 2, 64, 1, 65, 2, 66, 1),
    "table64": (1, 190, 1, 192, 1, 193, 2, 200, 1, 1, 1),
    "table128": (2, 384, 1, 385, 1, 1),
    "table256": (1, 768, 1, 769, 2, 1, 1, 1),
    "wide": (3, 3000, 3, 1, 1, 1, 1),
}


@pytest.mark.parametrize("block", ["64", "128", "256"])
@pytest.mark.parametrize("cbo,directed", [(0, False), (5, False), (0, True)])
@pytest.mark.parametrize("name", list(WIDTHS))
def test_levels_and_meeting_sets(name, cbo, directed, block, monkeypatch):
    monkeypatch.setenv("CENTRA_BIDIR_BLOCK", block)
    g = layers(WIDTHS[name], directed)
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g, count_bits_override=cbo)
        try:
            say(f"bidir {name} cbo {cbo} directed {directed} block {block}")
            off, nodes = binding.sample_paths(ctx, dg, 9, 1, 3, 1500, bidir=True)
            c_f, c_b = budgets(g, cbo)
            want_off, want_nodes = oracle.sample_paths_bidir(g, 9, 1, 3, 1500, c_f=c_f, c_b=c_b)
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
