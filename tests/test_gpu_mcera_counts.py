"""AMCERA trial sums against the oracle where the count kernel's spans end:
entry counts around whole batches of 64, spans of one batch and of several,
rows inside one span, on its edge and over many spans."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,hubs,t", [
    (7, 63, 1, 3), (64, 64, 0, 64), (200, 65, 2, 65), (3000, 5000, 3, 10), (5000, 1_048_576, 0, 5),
    (70_000, 1_048_577, 4, 9), (40, 2_200_000, 40, 2)])
def test_trial_sums(n, m, hubs, t):
    # one node per hyperedge: half of them hubs, so that rows of one entry and
    # of hundreds of thousands lie side by side
    rng = np.random.default_rng(m)
    nodes = rng.integers(0, n, m).astype(np.uint32)
    if hubs:
        half = rng.random(m) < 0.5
        nodes[half] = (rng.integers(0, hubs, int(half.sum())) * (n // hubs)).astype(np.uint32)
    off = np.arange(m + 1, dtype=np.uint64)
    say(f"trial sums n {n} entries {m} hubs {hubs} t {t}")
    ctx = binding.centra_create(0, 0)
    try:
        topk = torch.zeros(t, dtype=torch.int64, device="cuda")
        deg_topk = torch.zeros(1, dtype=torch.int64, device="cuda")
        b_max = torch.zeros(1, dtype=torch.int32, device="cuda")
        R = torch.zeros(n * t, dtype=torch.int32, device="cuda")
        binding.centra_mcera(ctx, n, torch.from_numpy(off.astype(np.int64)).cuda(),
                             torch.from_numpy(nodes.astype(np.int32)).cuda(), 11, 2, t, 3, topk, deg_topk, b_max, R)
        torch.cuda.synchronize()
        want = np.asarray(oracle.rade_sums(n, off, nodes, 11, 2, t))
        assert np.array_equal(R.cpu().numpy().reshape(want.shape), want)
    finally:
        binding.centra_destroy(ctx)
