"""Greedy cover in batches against the oracle: candidate sets that fit, that
tie in one bin and that exceed it, picks outside the first candidates, hubs
that share most of their samples, more nodes than columns, fewer positive
gains than rounds, lists of shared masks past their room."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding, inputs
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def uniform(n, m, lo, hi, rng):
    return [rng.choice(n, size=rng.integers(lo, hi + 1), replace=False) for _ in range(m)]


def hubs(n, m, h, rng):
    # every sample holds several of h hubs: gains fall together
    return [np.concatenate([rng.choice(h, size=rng.integers(1, 6), replace=False),
                            h + rng.choice(n - h, size=2, replace=False)]) for _ in range(m)]


SETS = {
    "flat": lambda rng: (50_000, uniform(50_000, 20_000, 1, 3, rng)),       # thousands of equal gains
    "few": lambda rng: (60_000, uniform(20, 30_000, 0, 2, rng)),            # 20 nodes of gain, k = 40
    "hubs": lambda rng: (45_000, hubs(45_000, 60_000, 200, rng)),
    "columns": lambda rng: (70_000, [np.unique(np.concatenate([16384 * rng.integers(0, 4, 2) + rng.integers(0, 3, 2),
                                                               rng.integers(0, 70_000, 1)])) for _ in range(40_000)]),
    "shared": lambda rng: (40_000, [np.arange(60)[rng.random(60) < 0.2] for _ in range(560_000)]),   # past the list
}


@pytest.mark.parametrize("k", [12, 40])
@pytest.mark.parametrize("name", list(SETS) + ["skewed"])
def test_matches_the_oracle(name, k):
    rng = np.random.default_rng(5)
    if name == "skewed":
        n = 200_000
        off, nodes = inputs.hyperedges(n, 150_000, 8, 3, 7)
    else:
        n, rows = SETS[name](rng)
        off = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.uint64)
        nodes = np.concatenate(rows).astype(np.uint32)
    say(f"greedy batches {name} k {k}: n {n} m {len(off) - 1} entries {int(off[-1])}")
    ctx = binding.centra_create(0, 0)
    try:
        o = torch.from_numpy(off.astype(np.int64)).cuda()
        v = torch.from_numpy(np.append(nodes, 0).astype(np.int32)).cuda()
        want_picks, want_cov = oracle.greedy_cover(n, off, nodes, k)
        for _ in range(2):
            picks = torch.zeros(k, dtype=torch.int32, device="cuda")
            cov = torch.zeros(k, dtype=torch.int64, device="cuda")
            n_picked = torch.zeros(1, dtype=torch.int32, device="cuda")
            binding.centra_greedy_cover(ctx, n, o, v, k, picks, cov, n_picked)
            torch.cuda.synchronize()
            got = int(n_picked.item())
            assert got == len(want_picks)
            assert picks.cpu().numpy()[:got].tolist() == list(want_picks)
            assert cov.cpu().numpy()[:got].tolist() == list(want_cov)
    finally:
        binding.centra_destroy(ctx)
