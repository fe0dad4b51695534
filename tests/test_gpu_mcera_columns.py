"""The AMCERA's selection over columns against the oracle: on either side of the
nodes one workgroup holds and of the values from which floors are taken, k
from one to more than the positive values, values in exact bins and in wide
ones, trials around groups of 64."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

SMALL = 36 << 10


def hyperedges(n, m, hub, rng):
    # two distinct nodes each, the first of them, for half the samples, one of `hub` hubs
    a = rng.integers(0, n, m)
    h = rng.random(m) < 0.5
    if hub:
        a[h] = rng.integers(0, hub, int(h.sum()))
    b = (a + 1 + rng.integers(0, n - 1, m)) % n
    return np.arange(0, 2 * m + 1, 2).astype(np.uint64), np.stack([a, b], 1).reshape(-1).astype(np.uint32)


@pytest.mark.parametrize("n,m,hub,t,k", [
    (2, 5, 0, 3, 2), (300, 40, 0, 65, 50), (1000, 200_000, 3, 10, 1), (SMALL, 60_000, 40, 5, 20),
    (SMALL + 1, 60_000, 40, 5, 20), (50_000, 3000, 0, 64, 4000), (60_000, 400_000, 5, 129, 7),
    (300_000, 500_000, 300, 112, 30), (600_000, 2000, 0, 60, 1000), (600_000, 2_000_000, 20, 57, 3)])
def test_column_sums(n, m, hub, t, k):
    off, nodes = hyperedges(n, m, hub, np.random.default_rng(n + t))
    say(f"columns n {n} m {m} hubs {hub} t {t} k {k}")
    ctx = binding.centra_create(0, 0)
    try:
        topk = torch.zeros(t, dtype=torch.int64, device="cuda")
        deg_topk = torch.zeros(1, dtype=torch.int64, device="cuda")
        b_max = torch.zeros(1, dtype=torch.int32, device="cuda")
        binding.centra_mcera(ctx, n, torch.from_numpy(off.astype(np.int64)).cuda(),
                             torch.from_numpy(nodes.astype(np.int32)).cuda(), 11, 2, t, k, topk, deg_topk, b_max)
        torch.cuda.synchronize()
        _, want, want_deg, want_b = oracle.mcera(n, off, nodes, 11, 2, t, k)
        assert np.array_equal(topk.cpu().numpy(), np.asarray(want))
        assert int(deg_topk.item()) == want_deg and int(b_max.item()) == want_b
    finally:
        binding.centra_destroy(ctx)
