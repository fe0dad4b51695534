"""Greedy cover by one workgroup: against the oracle at the edges of its rule
(state that just fits LDS and just does not, entries on either side of its
share per round), of its waves' 64-entry steps and of its unrolled walk, with
empty and long hyperedges."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

FIT = (144 << 10) // 4 - 2   # nodes whose gains, with 32 samples' bits, fill the state


@pytest.mark.parametrize("n,m,max_len,k", [
    (1, 1, 1, 1), (3, 70, 2, 5), (65, 63, 9, 65), (1025, 1025, 3, 7), (FIT, 32, 5, 3), (FIT + 1, 32, 5, 3),
    (5000, 20_000, 300, 4), (500, 12_288, 2, 1), (500, 12_289, 2, 1), (200, 5000, 40, 150)])
def test_matches_the_oracle(n, m, max_len, k):
    rng = np.random.default_rng(n + m)
    length = np.full(m, 1) if max_len == 2 and k == 1 else rng.integers(0, max_len + 1, m)
    rows = [np.unique(np.minimum((n * rng.random(int(x)) ** 2).astype(np.uint32), n - 1)) for x in length]
    off = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.uint64)
    nodes = np.concatenate(rows).astype(np.uint32)
    say(f"greedy n {n} m {m} entries {int(off[-1])} k {k}")
    ctx = binding.centra_create(0, 0)
    try:
        o = torch.from_numpy(off.astype(np.int64)).cuda()
        v = torch.from_numpy(np.append(nodes, 0).astype(np.int32)).cuda()
        picks = torch.zeros(k, dtype=torch.int32, device="cuda")
        cov = torch.zeros(k, dtype=torch.int64, device="cuda")
        n_picked = torch.zeros(1, dtype=torch.int32, device="cuda")
        binding.centra_greedy_cover(ctx, n, o, v, k, picks, cov, n_picked)
        torch.cuda.synchronize()
        want_picks, want_cov = oracle.greedy_cover(n, off, nodes, k)
        got = int(n_picked.item())
        assert got == len(want_picks)
        assert picks.cpu().numpy()[:got].tolist() == list(want_picks)
        assert cov.cpu().numpy()[:got].tolist() == list(want_cov)
    finally:
        binding.centra_destroy(ctx)
