"""GPU parity of centra_sample_paths where its level bitmap and its launch rule
change course: levels that end at and around word edges or span more than 64
words of the bitmap, levels of one node, and memory limits on either side of
the thread counts per BFS."""
import numpy as np
import pytest

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say

pytestmark = pytest.mark.gpu


def lantern(widths):
    # Undirected: one node, a layer of widths[0] nodes, one node, ... each
    # node joined to all of the neighbouring layers, so a BFS from an end has
    # exactly these level sizes; a tail of single nodes after it.
    layers, first = [], 0
    for w in [x for y in widths for x in (1, y)] + [1] * 70:
        layers.append(np.arange(first, first + w))
        first += w
    src = np.concatenate([np.repeat(a, len(b)) for a, b in zip(layers, layers[1:])])
    dst = np.concatenate([np.tile(b, len(a)) for a, b in zip(layers, layers[1:])])
    return inputs.from_edges(first, src, dst, directed=False)


@pytest.mark.parametrize("variant", ["hbm64", "hbm256"])
@pytest.mark.parametrize("widths", [(1, 62, 63, 64, 65), (9000,), (2, 4200, 3, 127, 128, 129)])
def test_level_starts(widths, variant, monkeypatch):
    monkeypatch.setenv("CENTRA_SAMPLER_VARIANT", variant)
    monkeypatch.setenv("CENTRA_WIDE", "0")
    g = lantern(widths)
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"level starts {widths} {variant}: 400 samples")
            off, nodes = binding.sample_paths(ctx, dg, 3, 1, 0, 400)
            want_off, want_nodes = oracle.sample_paths(g, 3, 1, 0, 400)
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)


@pytest.mark.parametrize("budget_mb,slots", [(1000, 2048), (2000, 3072), (4000, 1 << 30)])
def test_threads_per_bfs_follow_the_slots(budget_mb, slots):
    # budgets for fewer slots than 2,048 (256 threads each), than 3,072 (128
    # threads) and for more (64 threads)
    g = inputs.ba_graph(300, 5, 1)
    ctx = binding.centra_create(0, budget_mb << 20)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"budget {budget_mb} MB: 3000 samples")
            binding.centra_sampler_stats_get(ctx, reset=True)
            off, nodes = binding.sample_paths(ctx, dg, 7, 1, 0, 3000)
            st = binding.centra_sampler_stats_get(ctx)
            assert 1 <= st.slots < slots
            want_off, want_nodes = oracle.sample_paths(g, 7, 1, 0, 3000)
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
