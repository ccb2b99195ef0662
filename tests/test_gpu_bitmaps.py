"""GPU parity of the sampling phase on per-minibatch bitmaps, at the sizes where
its kernels change course: mask words of the list (32 and 64 minibatches), the
targets' placement (a workgroup for every 256 of them), the sampler's fanout bounds
and its wave-per-row form, chunks and runs beyond what one round locates, held and new
nodes beyond what LDS lists at once, list blocks of many entries, feature blocks
that span list blocks, node counts around a block and a range, and the first
shapes on either side of the limits where the radix sort takes over.  Every
output and statistic is compared with the oracle, element by element."""
import numpy as np
import pytest
import torch

import oracle
from tests.graphs import features
from tests.parity import compare_minibatch, feature_bytes, log
from tests.test_gpu_robustness import _failing_allocator

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def agnes():
    import paper_2601_01473_amd as ag
    return ag


def skewed_graph(n, deg, seed, heavy=0.3):
    """n nodes with 0 to 2 deg neighbours each (distinct, sorted), `heavy` of them among the first ids."""
    rng = np.random.default_rng(seed)
    d = rng.integers(0, 2 * deg + 1, size=n)
    rows = np.repeat(np.arange(n), d)
    few = max(1, min(n, 97))
    idx = np.where(rng.random(len(rows)) < heavy, rng.integers(0, few, len(rows)), rng.integers(0, n, len(rows)))
    key = np.unique(rows * np.int64(n) + idx)
    rows, idx = key // n, key % n
    off = np.zeros(n + 1, np.int64)
    np.add.at(off, rows + 1, 1)
    return np.cumsum(off), idx.astype(np.int32)


def check(ag, off, idx, targets, fan, dim=1, block=4096, dtype=np.float32, seed=11, mb=3, host=False):
    log("bitmaps", len(off) - 1, targets.shape, fan, "dim", dim, "block", block)
    feat = features(len(off) - 1, dim, 1, dtype)
    store = ag.Store(off, idx, feat, block)
    t = targets if host else torch.from_numpy(targets).cuda()
    batch = None
    o = oracle.Oracle(off, idx)
    fb = feature_bytes(feat)
    for step in range(2):                              # the second time with the batch's buffers
        batch = store.prepare(t, fan, seed=seed + step, mb_base=mb, batch=batch)
        got = batch.to_host()
        ref = o.hyperbatch(targets, fan, seed + step, mb)
        for j in range(targets.shape[0]):
            compare_minibatch(got[j], ref[j], oracle.gather(fb, ref[j].nodes), tag=(step, j))
        st = batch.stats()
        for k, v in oracle.hyperbatch_stats(off, block, fb.shape[1], ref, len(fan)).items():
            assert st[k] == v, (k, st[k], v)
    batch.close()
    store.close()


def draw_targets(n, H, B, seed):
    rng = np.random.default_rng(seed)
    return np.stack([rng.permutation(n)[:B] for _ in range(H)]).astype(np.int32)


@pytest.mark.parametrize("H", [1, 31, 32, 33, 64, 65, 127, 128, 129])
def test_minibatch_counts(agnes, H):
    off, idx = skewed_graph(700, 6, H)
    check(agnes, off, idx, draw_targets(700, H, 40, H), [5, 3], dim=3, block=64)


@pytest.mark.parametrize("B", [1, 2, 63, 1023, 1024, 1025, 2049, 4096, 4097])
def test_target_counts(agnes, B):
    off, idx = skewed_graph(5000, 5, 1)
    check(agnes, off, idx, draw_targets(5000, 2, B, B), [4, 2], host=True)


@pytest.mark.parametrize("f", [0, 1, 5, 6, 10, 11, 15, 16, 20, 21, 25, 26, 32, 33, 63, 64, 65, 129, 1024])
def test_fanouts(agnes, f):
    off, idx = skewed_graph(3000, 50, 2, heavy=0.5)
    check(agnes, off, idx, draw_targets(3000, 3, 50, f), [f, 3] if f > 40 else [7, f])


@pytest.mark.parametrize("n", [1, 2, 5, 511, 512, 513, 1025, 16383, 131073])
def test_node_counts(agnes, n):
    off, idx = skewed_graph(n, 4, 3)
    check(agnes, off, idx, draw_targets(n, 3, min(n, 300), n), [6, 4], dim=5, block=32)


@pytest.mark.parametrize("n", [(1 << 23) + 5, (1 << 24) + 1, (1 << 25) + 3])
def test_long_ranges(agnes, n):
    """Ranges of more than 2^17 nodes: 512 threads, and above 2^25 nodes more than
    64 KiB of LDS for the bits.  A range ends at its share of the weight, a 32nd
    or more (here even, so about as many nodes), or at the longest length, 2^18
    or 2^19 nodes: whichever comes first makes it long enough."""
    longest, need = (1 << 18, 1 << 17) if n <= 1 << 25 else (1 << 19, (65536 // 36) << 8)
    assert min(0.97 * n / 32, longest - 512) > need
    off, idx = skewed_graph(n, 1, 4, heavy=0.0)
    check(agnes, off, idx, draw_targets(n, 2, 600, 4), [3, 2, 2], dim=1, block=1 << 14)


def test_many_held_nodes_in_one_range(agnes):
    """All targets side by side: more held nodes in one range than LDS keeps."""
    n = 1 << 18
    off, idx = skewed_graph(n, 8, 5)
    t = np.stack([np.random.default_rng(j).permutation(4096) + 1000 for j in range(2)]).astype(np.int32)
    check(agnes, off, idx, t, [6, 3])


def test_many_new_nodes_in_one_range(agnes):
    """More new nodes in one range than k_bm_union lists at a time (2048): even
    weights make at most 33 ranges, so more than 33 x 2048 new nodes of a hop put
    more than 2048 into one of them, and more than 66 x 2048 call for a third window."""
    n, fan = 1 << 18, [15, 10]
    off, idx = skewed_graph(n, 20, 6, heavy=0.0)
    targets = draw_targets(n, 8, 4096, 6)         # (fewer would be left to the radix path)
    for m in oracle.Oracle(off, idx).hyperbatch(targets, fan, 11, 3):
        assert np.diff(m.layer_sizes).max() > 66 * 2048
    check(agnes, off, idx, targets, fan)


def test_more_chunks_than_one_round_locates(agnes):
    """Fanout 1024 makes chunks of four rows: over 256 of them per minibatch."""
    off, idx = skewed_graph(4000, 3, 7)
    check(agnes, off, idx, draw_targets(4000, 2, 1500, 7), [1024, 1024])


@pytest.mark.parametrize("dim,block", [(1, 1 << 14), (1, 16), (7, 64), (3, 1 << 12), (100, 1 << 15)])
def test_feature_blocks_and_list_blocks(agnes, dim, block):
    off, idx = skewed_graph(9000, 6, 8, heavy=0.8)
    check(agnes, off, idx, draw_targets(9000, 40, 100, 8), [8, 5], dim=dim, block=block)


def test_dense_list_blocks(agnes):
    """Every minibatch holds nearly every node: hundreds of entries per list block."""
    off, idx = skewed_graph(600, 30, 9)
    check(agnes, off, idx, draw_targets(600, 64, 300, 9), [20, 10], dim=2, block=256)


def test_wide_offsets(agnes, monkeypatch):
    monkeypatch.setenv("AGNES_WIDE_OFFSETS", "1")
    off, idx = skewed_graph(20000, 9, 10)
    check(agnes, off, idx, draw_targets(20000, 5, 200, 10), [40, 12, 3], dim=4, block=512)


def test_radix_path_keeps_its_shapes(agnes):
    """Past the limits (minibatches, targets): large sorts of the radix path."""
    off, idx = skewed_graph(1 << 21, 6, 11)
    check(agnes, off, idx, draw_targets(1 << 21, 6, 4100, 11), [9, 8], dim=1, block=4096)
    off, idx = skewed_graph(30000, 6, 12)
    check(agnes, off, idx, draw_targets(30000, 200, 64, 12), [9, 8], dim=1, block=4096)


def test_bad_targets_leave_the_batch_usable(agnes):
    off, idx = skewed_graph(2000, 5, 13)
    feat = features(2000, 4, 1)
    store = agnes.Store(off, idx, feat, 4096)
    good = draw_targets(2000, 4, 64, 13)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for bad, at in ((2000, (0, 0)), (-1, (3, 63)), (int(good[2, 5]), (2, 9))):
        t = good.copy()
        t[at] = bad
        b = store.begin(t, [5, 5], seed=1, stream=s1)
        with pytest.raises(agnes.AgnesError, match="target"):
            b.finish(stream=s2)
        b = store.begin(good, [5, 5], seed=1, batch=b, stream=s2)
        b.finish(stream=s1)
        got = b.to_host()
        ref = oracle.Oracle(off, idx).hyperbatch(good, [5, 5], 1, 0)
        for j in range(4):
            compare_minibatch(got[j], ref[j], oracle.gather(feature_bytes(feat), ref[j].nodes), tag=(bad, j))


def test_replay_on_a_store_that_takes_the_place_of_another(agnes):
    """A batch whose sampling was captured, on a second store of the same size at the
    first one's address but with other degrees, and so other node ranges."""
    n, fan = 5000, [6, 4]
    off, idx = skewed_graph(n, 6, 16, heavy=0.9)
    even = np.sort(np.random.default_rng(17).integers(0, n, len(idx)).astype(np.int32).reshape(-1))
    feat, t = features(n, 4, 1), draw_targets(n, 8, 100, 16)
    for attempt in range(8):
        first = agnes.Store(off, idx, feat, 4096)
        first.set_sampling_graph(True)
        b = None
        for step in range(3):
            b = first.prepare(t, fan, seed=step, batch=b)
        at = first.handle
        first.close()
        second = agnes.Store(off, even, feat, 4096)
        second.set_sampling_graph(True)
        log("second store", attempt, second.handle == at)
        if second.handle != at:
            b.close()
            second.close()
            continue
        for step in range(3):
            b = second.prepare(t, fan, seed=step, batch=b)
            got = b.to_host()
            ref = oracle.Oracle(off, even).hyperbatch(t, fan, step, 0)
            for j in range(8):
                compare_minibatch(got[j], ref[j], oracle.gather(feature_bytes(feat), ref[j].nodes), tag=(step, j))
        return
    pytest.skip("no second store at the first one's address")


def test_failing_finish_leaves_nothing_running(agnes):
    """The rows find no memory while the list is still being built on the sampling
    stream: when finish has raised, that stream is idle, and the batch may begin
    again on another one."""
    off, idx = skewed_graph(1 << 20, 6, 14)
    store = agnes.Store(off, idx, features(1 << 20, 1, 1), 4096)
    large, small = draw_targets(1 << 20, 128, 1024, 14), draw_targets(1 << 20, 3, 50, 15)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    state = {"calls": 0, "fail_at": -1}
    agnes.agnes_set_device_allocator(*_failing_allocator(agnes, state))
    try:
        for step in range(3):
            log("failing finish", step)
            b = store.begin(large, [10, 8], seed=step, stream=s1)
            state["fail_at"] = state["calls"]
            with pytest.raises(agnes.AgnesError, match="no memory"):
                b.finish(stream=s2)
            assert s1.query()
            b = store.begin(small, [5, 5], seed=1, batch=b, stream=s2).finish(stream=s1)
            got = b.to_host()
            ref = oracle.Oracle(off, idx).hyperbatch(small, [5, 5], 1, 0)
            for j in range(3):
                compare_minibatch(got[j], ref[j], tag=(step, j))
            b.close()
        store.close()
    finally:
        agnes.agnes_set_device_allocator(None, None)


@pytest.mark.parametrize("B,a,b", [(2, 0, 1), (257, 0, 256), (1024, 511, 1023), (1025, 0, 1024), (4096, 1024, 4095)])
def test_duplicate_targets_are_found_at_any_distance(agnes, B, a, b):
    n = 20000
    off, idx = skewed_graph(n, 4, 23)
    store = agnes.Store(off, idx, features(n, 4, 2), 4096)
    t = draw_targets(n, 2, B, 29)
    t[1, b] = t[1, a]
    with pytest.raises(agnes.AgnesError, match="twice"):
        store.prepare(t, [3], seed=1)
    t = np.ascontiguousarray(np.arange(2 * B, dtype=np.int32).reshape(2, B) * 2)      # consecutive hash slots
    got = store.prepare(t, [3], seed=1).to_host()
    ref = oracle.Oracle(off, idx).hyperbatch(t, [3], 1, 0)
    for j in range(2):
        assert np.array_equal(got[j]["nodes"], ref[j].nodes)
