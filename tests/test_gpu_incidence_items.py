"""The incidence (through the trial sums, which need every entry once) where the
build's item size changes and where buckets end inside items."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_03651_amd import binding
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries", [1, 1023, 1024, 1025, 196_608, 393_215, 393_216, 3_145_728])
@pytest.mark.parametrize("n", [2047, 2049, 12_287, 12_288, 12_289])
def test_every_entry_once(n, entries):
    rng = np.random.default_rng(entries)
    nodes = np.minimum((n * rng.random(entries) ** 4).astype(np.uint32), n - 1)
    off = np.arange(entries + 1, dtype=np.uint64)
    say(f"incidence n {n} entries {entries}")
    ctx = binding.centra_create(0, 0)
    try:
        topk = torch.zeros(3, dtype=torch.int64, device="cuda")
        deg_topk = torch.zeros(1, dtype=torch.int64, device="cuda")
        b_max = torch.zeros(1, dtype=torch.int32, device="cuda")
        R = torch.zeros(n * 3, dtype=torch.int32, device="cuda")
        binding.centra_mcera(ctx, n, torch.from_numpy(off.astype(np.int64)).cuda(),
                             torch.from_numpy(nodes.astype(np.int32)).cuda(), 5, 1, 3, 4, topk, deg_topk, b_max, R)
        torch.cuda.synchronize()
        want = np.asarray(oracle.rade_sums(n, off, nodes, 5, 1, 3))
        assert np.array_equal(R.cpu().numpy().reshape(want.shape), want)
        assert int(deg_topk.item()) == int(np.sort(np.bincount(nodes, minlength=n))[-4:].sum())
    finally:
        binding.centra_destroy(ctx)
