"""GPU parity of the row copy at row widths that are no multiple of 16 bytes
(16-byte pieces at 4-byte boundaries, the last one overlapping the one before
it), and of a batch reused with growing and shrinking hyperbatches and invalid
targets between."""
import numpy as np
import pytest
import torch

import oracle
from tests.graphs import features, random_graph
from tests.parity import compare_minibatch, feature_bytes, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def agnes():
    import paper_2601_01473_amd as ag
    return ag


def draw_targets(n, H, B, seed):
    rng = np.random.default_rng(seed)
    return np.stack([rng.permutation(n)[:B] for _ in range(H)]).astype(np.int32)


def compare(batch, off, idx, feat, t, fan, seed):
    got = batch.to_host()
    ref = oracle.Oracle(off, idx).hyperbatch(t, fan, seed, 0)
    fb = feature_bytes(feat)
    for j in range(t.shape[0]):
        compare_minibatch(got[j], ref[j], oracle.gather(fb, ref[j].nodes), tag=(t.shape, j))


@pytest.mark.parametrize("dim", [1, 2, 3, 4, 5, 7, 8, 9, 17, 31, 33, 63, 75, 129, 255, 257, 513, 1025])
@pytest.mark.parametrize("unroll", [0, 8, 16])
def test_row_widths(agnes, dim, unroll):
    log("row width", dim * 4, "unroll", unroll)
    off, idx = random_graph(400, 6, 1)
    feat = features(400, dim, dim)
    store = agnes.Store(off, idx, feat, 8192)
    store.set_gather_shape(unroll=unroll, nontemporal=unroll != 8)
    t = draw_targets(400, 5, 40, dim)
    b = store.prepare(t, [4, 3], seed=2)
    compare(b, off, idx, feat, t, [4, 3], 2)
    staged = agnes.Store(off, idx, feat, 8192, pool_blocks=3)
    compare(staged.prepare(t, [4, 3], seed=2), off, idx, feat, t, [4, 3], 2)


@pytest.mark.parametrize("profiled", [False, True])
@pytest.mark.parametrize("dim", [3, 64, 1500])
def test_prepare_with_a_reused_batch(agnes, dim, profiled):
    """Rows beyond the buffer (growing), within it (shrinking), and bad targets between."""
    n = 30000
    off, idx = random_graph(n, 5, 3, hubs=1, hub_deg=50)
    feat = features(n, dim, 4)
    store = agnes.Store(off, idx, feat, 8192)
    store.set_profiling(profiled)
    batch = None
    for step, (H, B) in enumerate([(2, 30), (3, 200), (3, 100), (8, 600), (1, 5), (8, 600)]):
        log("reused", dim, H, B)
        t = draw_targets(n, H, B, step)
        if step == 3:
            bad = t.copy()
            bad[1, 2] = bad[1, 3]
            with pytest.raises(agnes.AgnesError, match="twice"):
                store.prepare(bad, [6, 4], seed=step, batch=batch)
            batch = None
        batch = store.prepare(t, [6, 4], seed=step, batch=batch)
        compare(batch, off, idx, feat, t, [6, 4], step)
        s = batch.stats()
        assert (s["gather_ms"] >= 0) == profiled and (s["sample_ms"] >= 0) == profiled


def test_prepare_then_forward_and_pipelined_calls(agnes):
    """The same batch through prepare, then begin / finish on other streams."""
    off, idx = random_graph(5000, 6, 5)
    feat = features(5000, 32, 6)
    store = agnes.Store(off, idx, feat, 4096)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    batch = None
    for step in range(4):
        t = draw_targets(5000, 4, 50 + 100 * step, step)
        if step % 2 == 0:
            batch = store.prepare(t, [5, 5], seed=step, batch=batch, stream=s1)
        else:
            batch = store.begin(t, [5, 5], seed=step, batch=batch, stream=s2).finish(stream=s1)
        compare(batch, off, idx, feat, t, [5, 5], step)
