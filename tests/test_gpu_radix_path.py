"""The radix sort and merge-path join on small shapes, which bitmaps serve by
default: the parity, replay, stream, allocator and staged-tier tests once more on
stores built with AGNES_RADIX_JOIN=1."""
import numpy as np
import pytest
import torch

from tests.graphs import distinct_targets, features, random_graph
from tests.test_gpu_bitmaps import check, draw_targets
from tests.test_gpu_parity import (  # noqa: F401
    agnes, test_argument_limits_are_rejected_and_store_stays_usable, test_determinism_reuse_and_grouping,
    test_eight_hops, test_fanout_register_paths, test_finish_on_other_stream_and_errors,
    test_invalid_targets_are_rejected_and_store_stays_usable, test_isolated_and_single_node_graph,
    test_large_fanout_memory_path, test_largest_fanout_against_a_hub, test_multigraph_rows,
    test_random_graph_int32_offsets_fp16, test_random_graphs_int64, test_random_graphs_int64_kept_wide_on_device,
    test_runs_spanning_join_tiles, test_sampling_graph_replays_equal_launches, test_stored_fixture_on_gpu,
    test_three_batches_two_sampling_streams_one_gather_stream, test_torch_allocator_owns_device_memory,
    test_two_batches_in_flight_on_two_streams, test_zero_fanout_and_take_all)
from tests.test_gpu_robustness import _failing_allocator
from tests.test_gpu_staging import (  # noqa: F401
    test_feature_cache_matches_oracle_and_model, test_staged_tier_batches_in_flight_on_several_streams)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def radix(monkeypatch):
    monkeypatch.setenv("AGNES_RADIX_JOIN", "1")


def test_the_switch_selects_the_path(agnes, monkeypatch):
    """The paths ask for different buffers (the radix sort for its four and its
    histograms): a batch's first hyperbatch shows which one ran."""
    off, idx = random_graph(2000, 8, seed=1)
    feat, t = features(2000, 4, 1), distinct_targets(2000, 3, 40, 2)
    state = {"calls": 0, "fail_at": -1}
    asked = {}
    agnes.agnes_set_device_allocator(*_failing_allocator(agnes, state))
    try:
        for switch in ("0", "1", "0"):
            monkeypatch.setenv("AGNES_RADIX_JOIN", switch)
            store = agnes.Store(off, idx, feat, 4096)
            state["calls"] = 0
            b = store.prepare(t, [4, 3], seed=1)
            asked.setdefault(switch, []).append(state["calls"])
            b.close()
            store.close()
    finally:
        agnes.agnes_set_device_allocator(None, None)
    torch.cuda.synchronize()
    assert asked["0"][0] == asked["0"][1] != asked["1"][0]


@pytest.mark.parametrize("H,B,fan,left", [(1, 4096, [20, 15, 10], True), (2, 4096, [50, 50], True),
                                          (1, 4096, [10, 5], False), (16, 1024, [20, 15, 10], False)])
def test_few_large_minibatches_are_left_to_it(agnes, monkeypatch, H, B, fan, left):
    """By default, too: they ask for the radix path's buffers, with the oracle's results."""
    n = 1 << 16
    off = np.arange(n + 1, dtype=np.int64) * 40
    idx = np.sort(np.random.default_rng(3).integers(0, n, (n, 40)), axis=1).astype(np.int32).ravel()
    t = draw_targets(n, H, B, 4)
    state = {"calls": 0, "fail_at": -1}
    asked = []
    agnes.agnes_set_device_allocator(*_failing_allocator(agnes, state))
    try:
        for switch in ("0", "1"):
            monkeypatch.setenv("AGNES_RADIX_JOIN", switch)
            store = agnes.Store(off, idx, features(n, 1, 1), 4096)
            state["calls"] = 0
            b = store.prepare(t, fan, seed=1)
            asked.append(state["calls"])
            b.close()
            store.close()
    finally:
        agnes.agnes_set_device_allocator(None, None)
    assert (asked[0] == asked[1]) == left
    monkeypatch.setenv("AGNES_RADIX_JOIN", "0")
    check(agnes, off, idx, t, fan)
