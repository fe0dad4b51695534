"""The threads per BFS of stream-ordered launches, seen by the memory that their
slots take (4,096 of one wave, 2,048 of 128 threads): by the longest row of the
graph, with the oracle's hyperedges."""
import numpy as np
import pytest
import torch

from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import oracle_paths, say
from tests.test_gpu_fused_threads import star

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,slots", [("ba", 4096), ("star", 2048)])
def test_append(kind, slots):
    n, count, cap = 4000, 40_000, 40_000 * 16
    g = inputs.ba_graph(n, 4, 7) if kind == "ba" else star(n)
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"append, {kind}: {count} samples")
            off = torch.zeros(count + 1, dtype=torch.int64, device="cuda")
            nodes = torch.zeros(cap, dtype=torch.int32, device="cuda")
            free = torch.cuda.mem_get_info()[0]
            binding.centra_reserve(ctx, dg.handle, n, count, count, cap, 5, 0)
            taken = free - torch.cuda.mem_get_info()[0]
            state = 20.125 * n + 12 * 65536   # bytes of a slot
            say(f"  {taken / state:.0f} slots' worth taken")
            assert 0.9 * slots * state < taken < 1.5 * slots * state
            binding.centra_sample_paths_append(ctx, dg.handle, 7, 1, 0, count, off, nodes)
            assert binding.centra_check(ctx) == 0
            o, v = off.cpu().numpy(), nodes.cpu().numpy()
            for i, w in enumerate(oracle_paths(g, 7, 1, range(0, 200), dg.info()[1])):
                assert np.array_equal(v[int(o[i]):int(o[i + 1])].astype(np.uint32), w[0])
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
