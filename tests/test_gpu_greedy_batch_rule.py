"""Greedy cover where the batches give up: candidates' rows on either side of
the entries per round and of the entries per sample, rows too long only in a
later batch, hyperedges that name a node twice.  Against the oracle, and the
rounds alone (few rounds) against the same rounds of a larger call."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

N = 45_000   # one workgroup's state does not fit LDS


def cover(n, off, nodes, k):
    ctx = binding.centra_create(0, 0)
    try:
        o = torch.from_numpy(off.astype(np.int64)).cuda()
        v = torch.from_numpy(np.append(nodes, 0).astype(np.int32)).cuda()
        picks = torch.zeros(k, dtype=torch.int32, device="cuda")
        cov = torch.zeros(k, dtype=torch.int64, device="cuda")
        n_picked = torch.zeros(1, dtype=torch.int32, device="cuda")
        binding.centra_greedy_cover(ctx, n, o, v, k, picks, cov, n_picked)
        torch.cuda.synchronize()
        got = int(n_picked.item())
        return picks.cpu().numpy()[:got].tolist(), cov.cpu().numpy()[:got].tolist()
    finally:
        binding.centra_destroy(ctx)


def exactly(m, entries, hubs, rng):
    """m samples over hubs nodes, all of which are candidates, entries in all."""
    length = np.full(m, entries // m)
    length[:entries - int(length.sum())] += 1
    return [rng.choice(hubs, size=int(x), replace=False) for x in rng.permutation(length)]


def later(rng):
    """10 nodes of 10,000 samples each, then 200 of 2,000 each in one bin."""
    rows = [np.array([u]) for u in range(10) for _ in range(10_000)]
    return rows + [np.array([10 + u]) for u in range(200) for _ in range(2000)]


CASES = {
    "entries at": (12, lambda rng: exactly(80_000, 12 * 12288, 40, rng)),
    "entries past": (12, lambda rng: exactly(80_000, 12 * 12288 + 1, 40, rng)),
    "overlap at": (12, lambda rng: exactly(2000, 4000, 40, rng)),
    "overlap past": (12, lambda rng: exactly(2000, 4001, 40, rng)),
    "dense": (40, lambda rng: exactly(3000, 60_000, 60, rng)),
    "later": (16, later),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rows_too_long(name):
    k, make = CASES[name]
    rows = make(np.random.default_rng(3))
    off = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.uint64)
    nodes = np.concatenate(rows).astype(np.uint32)
    say(f"greedy batch rule {name} k {k}: m {len(rows)} entries {int(off[-1])}")
    picks, cov = cover(N, off, nodes, k)
    want_picks, want_cov = oracle.greedy_cover(N, off, nodes, k)
    assert picks == list(want_picks)
    assert cov == list(want_cov)


@pytest.mark.parametrize("k", [12, 40])
def test_a_node_twice_in_a_hyperedge(k):
    rng = np.random.default_rng(9)
    rows = [rng.choice(N, size=3, replace=False) for _ in range(20_000)]
    for i in range(0, 20_000, 7):   # node i % 50 twice, among the candidates
        rows[i] = np.array([i % 50, i % 50, 50 + i])
    off = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.uint64)
    nodes = np.concatenate(rows).astype(np.uint32)
    say(f"greedy batch, a node twice, k {k}")
    picks, cov = cover(N, off, nodes, k)
    few_picks, few_cov = cover(N, off, nodes, 11)   # rounds from the start
    want_picks, _ = oracle.greedy_cover(N, off, nodes, k)
    assert picks == list(want_picks)
    assert picks[:11] == few_picks
    assert cov[:11] == few_cov
