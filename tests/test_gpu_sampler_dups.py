"""GPU parity of centra_sample_paths on searches whose rounds are full of arcs
to nodes already reached: dense layers, where a round may bring as many
different such nodes as its table of duplicates takes, with node ids that
share filter bits (so that some of them are new after all) and without."""
import numpy as np
import pytest

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say

pytestmark = pytest.mark.gpu


def layers(widths, n):
    # neighbouring layers joined completely, ids spread at random over n nodes
    rng = np.random.default_rng(sum(widths))
    ids = np.split(rng.permutation(n)[:sum(widths)], np.cumsum(widths)[:-1])
    src = np.concatenate([np.repeat(a, len(b)) for a, b in zip(ids, ids[1:])])
    dst = np.concatenate([np.tile(b, len(a)) for a, b in zip(ids, ids[1:])])
    # the other nodes hang on the layers one by one, so that every pair is joined
    rest = np.setdiff1d(np.arange(n), np.concatenate(ids))
    on = np.concatenate(ids)[rng.integers(0, sum(widths), len(rest))]
    return inputs.from_edges(n, np.concatenate([src, rest]), np.concatenate([dst, on]), directed=False)


@pytest.mark.parametrize("variant", ["hbm64", "hbm128", "hbm256", "hbm512"])
@pytest.mark.parametrize("widths,n,c_bits", [
    ((1, 190, 65, 257, 300, 1), 1000, 0), ((40, 512, 400, 300, 60), 3000, 6), ((3, 700, 700, 700, 200), 40_000, 0),
    ((2, 1030, 520, 1030), 70_000, 9)])
def test_rounds_of_duplicates(widths, n, c_bits, variant, monkeypatch):
    monkeypatch.setenv("CENTRA_SAMPLER_VARIANT", variant)
    monkeypatch.setenv("CENTRA_WIDE", "0")
    g = layers(widths, n)
    count = 300
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g, count_bits_override=c_bits)
        try:
            say(f"duplicates {widths} of {n} nodes, count bits {c_bits or 'full'}, {variant}: {count} samples")
            off, nodes = binding.sample_paths(ctx, dg, 9, 2, 0, count)
            want_off, want_nodes = oracle.sample_paths(g, 9, 2, 0, count, c_bits=dg.info()[1])
            assert np.array_equal(off_np(off), want_off)
            assert np.array_equal(nodes_np(nodes), want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
