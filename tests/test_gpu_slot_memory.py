"""The per-BFS state of both path samplers where memory does not hold as much
of it as a launch has a use for."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, oracle_paths, say

pytestmark = pytest.mark.gpu


def draw(call, ctx, dg, count, per=64):
    off = torch.zeros(count + 1, dtype=torch.int64, device="cuda")
    nodes = torch.zeros(count * per, dtype=torch.int32, device="cuda")
    binding.centra_sampler_stats_get(ctx, reset=True)
    call(ctx, dg.handle, 7, 1, 0, count, off, nodes, None, None, None)
    torch.cuda.synchronize()
    return off_np(off), nodes_np(nodes), binding.centra_sampler_stats_get(ctx)


def test_both_samplers_on_one_context():
    # node counts at which the two states together would take the whole device
    n, count = 2_100_000, 16_384
    g = inputs.ba_graph(n, 2, 9)
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            total = torch.cuda.mem_get_info()[1]
            say(f"both samplers, n {n}: {count} samples each")
            off, nodes, st = draw(binding.centra_sample_paths, ctx, dg, count)
            boff, bnodes, bst = draw(binding.centra_sample_paths_bidir, ctx, dg, count)
            left = torch.cuda.mem_get_info()[0]
            say(f"  slots {st.slots} and {bst.slots}, {left / 1e9:.1f} of {total / 1e9:.1f} GB left")
            assert st.slots >= 1 and bst.slots >= 1 and left > total // 32
            c = dg.info()[1]
            for i, w in enumerate(oracle_paths(g, 7, 1, range(0, 4), c)):
                assert np.array_equal(nodes[int(off[i]):int(off[i + 1])], w[0])
            want_off, want_nodes = oracle.sample_paths_bidir(g, 7, 1, 0, 4)
            assert np.array_equal(boff[:5], want_off)
            assert np.array_equal(bnodes[:int(want_off[-1])], want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
