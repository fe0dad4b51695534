"""centra_reserve covers every call up to the sizes it was given: extensions
with fewer trials and appends of fewer samples afterwards take no device
memory (the workspaces of neither grow with every size)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import nodes_np, off_np, say, to_dev_u32, to_dev_u64

pytestmark = pytest.mark.gpu


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("t_max", [65, 100, 200])
def test_fewer_trials_than_reserved(t_max):
    n, m, k = 300_000, 20_000, 5
    off, nodes = inputs.hyperedges(n, m, 6, 3, 2)
    d_off, d_nodes = to_dev_u64(off), to_dev_u32(nodes)
    pk = torch.zeros(k, dtype=torch.int32, device="cuda")
    cv = torch.zeros(k, dtype=torch.int64, device="cuda")
    one = [torch.zeros(1, dtype=x, device="cuda") for x in (torch.int32, torch.int64, torch.int32)]
    topk = torch.zeros(t_max, dtype=torch.int64, device="cuda")
    trials = [x for x in (1, 64, 65, 128, 192) if x < t_max] + [t_max]
    say(f"reserve for {t_max} trials, extensions with {trials}")
    for run in range(2):   # (the first loads the kernels)
        ctx = binding.centra_create(0, 0)
        try:
            binding.centra_reserve(ctx, None, n, 0, m, len(nodes), k, t_max)
            before = free_bytes()
            for t in trials:
                binding.centra_extend(ctx, n, k, 0, m, d_off, d_nodes, None, pk, cv, one[0], t, 3, 1, topk, one[1],
                                      one[2])
                if run:
                    assert free_bytes() == before, f"t = {t}"
                    _, wtop, wdk, _ = oracle.mcera(n, off, nodes, 3, 1, t, k)
                    assert np.array_equal(topk.cpu().numpy()[:t], wtop) and int(one[1].item()) == wdk
            assert binding.centra_check(ctx) == binding.CENTRA_OK
        finally:
            binding.centra_destroy(ctx)


@pytest.mark.parametrize("kind", ["ba", "grid"])
def test_fewer_samples_than_reserved(kind):
    # batches on both sides of the sample counts at which the threads per BFS change
    g = inputs.ba_graph(5000, 4, 3) if kind == "ba" else inputs.grid_graph(20)
    batches = [20_000, 16_383, 2048, 2047, 300, 1]
    total = sum(batches)
    w_off, w_nodes = oracle.sample_paths(g, 5, 2, 0, total)
    cap = int(w_off[-1])
    say(f"reserve for {batches[0]} samples of {kind}, appends of {batches}")
    for run in range(2):
        ctx = binding.centra_create(0, 0)
        dg = binding.DeviceGraph(ctx, g)
        try:
            off = torch.zeros(total + 1, dtype=torch.int64, device="cuda")
            nodes = torch.zeros(cap, dtype=torch.int32, device="cuda")
            binding.centra_reserve(ctx, dg.handle, g.n, batches[0], total, cap, 0, 0)
            before, m = free_bytes(), 0
            for c in batches:
                binding.centra_sample_paths_append(ctx, dg.handle, 5, 2, m, c, off[m:], nodes, cap)
                m += c
                if run:
                    assert free_bytes() == before, f"{c} samples"
            assert binding.centra_check(ctx) == binding.CENTRA_OK
            assert np.array_equal(off_np(off), w_off) and np.array_equal(nodes_np(nodes), w_nodes)
        finally:
            dg.release()
            binding.centra_destroy(ctx)
