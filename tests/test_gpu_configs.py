"""GPU parity on the five synthetic workloads at full size.

Node ids and per-hop CSR are compared with the CPU oracle element by element for
every minibatch of the hyperbatch, together with the exact statistics.  Feature
bytes are compared with the oracle's gather on a sample of minibatches, and for
every output row through the defining property out[i] == X[nodes[i]], checked
on the device with torch's own index_select.

The launch configuration is the one the benchmark times (one prepare call on
the current stream, batch reuse).
"""
import ctypes
import time

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import compare_minibatch, feature_bytes, log

pytestmark = pytest.mark.gpu


def gather_property_on_device(ag, store_feat_host: np.ndarray, batch) -> None:
    """out[i] == X[nodes[i]] for every gathered row, via torch.index_select on the GPU."""
    v = batch.view()
    H = v.H
    rows = int(np.ctypeslib.as_array(v.node_off, shape=(H + 1,))[H])
    rb = v.row_bytes
    words = rb // 4
    X = torch.from_numpy(feature_bytes(store_feat_host).view(np.int32).reshape(-1, words)).cuda()
    nodes = torch.empty(rows, dtype=torch.int32, device="cuda")
    out = torch.empty((rows, words), dtype=torch.int32, device="cuda")
    hip = ag._hiprt()
    torch.cuda.synchronize()
    assert hip.hipMemcpy(ctypes.c_void_p(nodes.data_ptr()), ctypes.c_void_p(v.nodes), rows * 4, 3) == 0
    assert hip.hipMemcpy(ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(v.features), rows * rb, 3) == 0
    chunk = 1 << 20
    for a in range(0, rows, chunk):
        ref = torch.index_select(X, 0, nodes[a:a + chunk].long())
        assert torch.equal(ref, out[a:a + chunk]), ("feature rows differ in chunk", a)
    del X, out, nodes
    torch.cuda.empty_cache()


def run_config(ag, name, H=None, feature_sample=4):
    cfg = synth.CONFIGS[name]
    t0 = time.time()
    w = synth.workload(cfg, H=H)
    log(f"[{name} H={w['H']}] inputs ready in {time.time() - t0:.1f}s: E={len(w['indices'])}")
    store = ag.Store(w["offsets"], w["indices"], w["features"], cfg.block_bytes,
                     feat_dtype=cfg.feat_dtype)
    log(f"[{name}] store built")
    t = torch.from_numpy(w["targets"]).cuda()
    b = store.prepare(t, cfg.fanouts, seed=cfg.seed)            # warm-up call (allocations)
    b = store.prepare(t, cfg.fanouts, seed=cfg.seed, batch=b)   # the call the benchmark times
    torch.cuda.synchronize()
    log(f"[{name}] prepared: {b.stats()}")
    got = b.to_host(features=False)
    o = oracle.Oracle(w["offsets64"], w["indices"])
    ref = o.hyperbatch(w["targets"], cfg.fanouts, cfg.seed, 0)
    log(f"[{name}] oracle done")
    Hh = w["H"]
    fb = feature_bytes(w["features"])
    sample = sorted(set(np.linspace(0, Hh - 1, min(feature_sample, Hh)).astype(int).tolist()))
    for j in range(Hh):
        compare_minibatch(got[j], ref[j], None, tag=(name, j))
    feats = b.to_host(minibatches=sample)
    for k, j in enumerate(sample):
        compare_minibatch(feats[k], ref[j], oracle.gather(fb, ref[j].nodes), tag=(name, "feat", j))
    st = b.stats()
    want = oracle.hyperbatch_stats(w["offsets64"], cfg.block_bytes, cfg.row_bytes, ref, len(cfg.fanouts))
    for k, v in want.items():
        assert st[k] == v, (name, k, st[k], v)
    gather_property_on_device(ag, w["features"], b)
    log(f"[{name}] parity ok")
    b.close()
    store.close()
    torch.cuda.empty_cache()


@pytest.fixture(scope="module")
def agnes():
    import paper_2601_01473_amd as ag
    return ag


def test_config_c1(agnes):
    run_config(agnes, "c1", feature_sample=8)


def test_config_c2(agnes):
    run_config(agnes, "c2")


def test_config_c3(agnes):
    run_config(agnes, "c3")


def test_config_c4(agnes):
    run_config(agnes, "c4")


@pytest.mark.parametrize("H", [1, 8, 64, 256])
def test_config_c5_hyperbatch_sweep(agnes, H):
    run_config(agnes, "c5", H=H)


@pytest.mark.parametrize("radix", [False, True])
def test_config_c2_with_64_minibatches(agnes, radix, monkeypatch):
    """C2's graph (20-bit node ids: two radix passes of 10-bit digits) with 64
    minibatches: the last hop's bound (64 x 16384 x 10 edges) is above 8M keys,
    where 8-bit digits would take 8192-key tiles; on the radix path 10-bit
    digits keep 4096.  The default path takes bitmaps."""
    monkeypatch.setenv("AGNES_RADIX_JOIN", "1" if radix else "0")
    run_config(agnes, "c2", H=64)
