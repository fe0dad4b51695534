"""The per-BFS state of both path samplers where memory does not hold as much
of it as a launch has a use for: a budget or a filled device gives fewer
slots, and a later call of the same kind keeps them."""
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


@pytest.mark.parametrize("bidir", [False, True])
@pytest.mark.parametrize("share", [1.1, 0.9, 0.4, 0.001])
def test_slots_cut_by_the_budget_are_kept(bidir, share, monkeypatch):
    # shares of the state of as many slots as half of the device may hold; the
    # smallest leaves room for one or two
    monkeypatch.setenv("CENTRA_SAMPLER_VARIANT", "hbm64")
    n, count = (1_000_000, 20_000) if share > 0.01 else (3000, 400)
    g = inputs.ba_graph(n, 3, 5)
    state = 1792 * 40 * n if bidir else 3072 * (20.125 * n + 12 * 65536)
    call = binding.centra_sample_paths_bidir if bidir else binding.centra_sample_paths
    ctx = binding.centra_create(0, int(share * state) + (64 << 20 if n > 3000 else 1 << 20))
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            say(f"bidir {bidir}, budget for {share} of the slots: {count} samples three times")
            got = [draw(call, ctx, dg, count) for _ in range(3)]
            say("  slots", [x[2].slots for x in got])
            for off, nodes, st in got[1:]:
                assert st.slots == got[0][2].slots >= 1
                assert np.array_equal(off, got[0][0]) and np.array_equal(nodes, got[0][1])
            if n > 3000:   # halves of the most that may take half of the device
                assert got[0][2].slots == ({1.1: 1792, 0.9: 896, 0.4: 448} if bidir else
                                           {1.1: 3072, 0.9: 1536, 0.4: 768})[share]
            if not bidir:
                want = oracle_paths(g, 7, 1, range(0, 40), dg.info()[1])
                off, nodes = got[0][:2]
                assert all(np.array_equal(nodes[int(off[i]):int(off[i + 1])], w[0]) for i, w in enumerate(want))
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)


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


@pytest.mark.parametrize("paths_before", [False, True])
def test_bidirectional_slots_beyond_the_lean_count(paths_before):
    # the slots that hide its latency at a million nodes, whose state is close
    # to half of the device, or as many as leave a quarter of it free
    n, count = 1_000_000, 20_000
    g = inputs.ba_graph(n, 2, 9)
    ctx = binding.centra_create(0, 0)
    try:
        dg = binding.DeviceGraph(ctx, g)
        try:
            if paths_before:   # 4,096 slots of the path sampler beside them
                draw(binding.centra_sample_paths, ctx, dg, 40_000)
            torch.cuda.empty_cache()
            free, total = torch.cuda.mem_get_info()
            off, nodes, st = draw(binding.centra_sample_paths_bidir, ctx, dg, count)
            say(f"bidir, n {n}: {st.slots} slots, {free / 1e9:.1f} of {total / 1e9:.1f} GB free before")
            room = min(total // 32 * 15, free - (1 << 30) - total // 4)
            assert st.slots >= min(3584, max(1792, room // (40 * n) - 1))
            want_off, want_nodes = oracle.sample_paths_bidir(g, 7, 1, 0, 4)
            assert np.array_equal(off[:5], want_off)
            assert np.array_equal(nodes[:int(want_off[-1])], want_nodes)
        finally:
            dg.release()
    finally:
        binding.centra_destroy(ctx)
