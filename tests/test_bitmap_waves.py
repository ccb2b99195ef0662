"""The kernels of the bitmap path on the CPU (host_waves/waves.cpp), element by
element against the oracle, with a workgroup's waves run lowest first and highest
first between its barriers: a result that depends on the order shows an access
that no barrier orders.  Every wave-wide exchange must be reached by a whole wave,
and every buffer of the library's size ends at memory that cannot be accessed."""
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
from tests.graphs import distinct_targets, random_graph

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2601_01473_amd", "csrc")


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    d = tmp_path_factory.mktemp("waves")
    text = open(os.path.join(CSRC, "bitmap.hip")).read()
    src, exe = d / "bitmap_host.inc", d / "waves"
    # static arrays are the workgroup's (one runs at a time), dynamic ones are in waves.cpp
    src.write_text(re.sub(r"\b__shared__\b", "static", re.sub(r"\bextern __shared__\b", "extern", text)))
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-fno-strict-aliasing", "-DBITMAP_SOURCE=\"%s\"" % src,
                        "-I" + os.path.join(HERE, "host_waves"), "-I" + CSRC, os.path.join(HERE, "host_waves", "waves.cpp"),
                        "-o", str(exe)], capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stderr

    def run(off, idx, targets, fan, bounds, seed, mb, highest_first, rpb=16, e_blk_log2=5):
        n, (H, B), L = len(off) - 1, targets.shape, len(fan)
        # list blocks: whole feature blocks, and a cut at every range
        cuts = sorted(set(range(0, n, 4 * rpb)) | set(bounds)) + ([n] if bounds[-1] != n else [])
        first = [cuts.index(b) for b in bounds]
        with open(d / "in", "wb") as f:
            for x, t in (([n, len(idx), H, B, L, len(bounds) - 1, len(cuts) - 1, rpb, e_blk_log2, seed, mb,
                           highest_first], np.int64), (fan, np.int32), (off, np.int64), (idx, np.int32),
                         (targets, np.int32), (bounds + first, np.int32), (cuts, np.int32)):
                np.asarray(x, t).tofile(f)
        r = subprocess.run([str(exe), str(d / "in"), str(d / "out")], capture_output=True, text=True, env=env,
                           timeout=300)
        assert r.returncode == 0, r.stderr
        data, at = (d / "out").read_bytes(), [0]

        def take(count, t):
            x = np.frombuffer(data, t, count, at[0])
            at[0] += x.nbytes
            return x

        out = dict(err=take(H, np.uint32), sizes=take(H * (L + 1), np.int32).reshape(H, L + 1),
                   edges=take(H * L, np.int64).reshape(H, L))
        rows = int(out["sizes"][:, L].sum())
        out["nodes"], out["list_key"], out["list_val"] = take(rows, np.int32), take(rows, np.uint64), take(rows, np.int32)
        out["stats"] = take(2 + L, np.int64)
        out["row_ptr"], out["col"] = [], []
        for l in range(L):
            out["row_ptr"].append(take(int(out["sizes"][:, l].sum()) + H, np.int32))
            out["col"].append(take(int(out["edges"][:, l].sum()), np.int32))
        assert at[0] == len(data)
        return out

    def plan(off, idx, H, B, fan, K=33):
        with open(d / "in", "wb") as f:
            for x, t in (([len(off) - 1, len(idx), H, B, len(fan), K], np.int64), (fan, np.int32), (off, np.int64),
                         (idx, np.int32)):
                np.asarray(x, t).tofile(f)
        r = subprocess.run([str(exe), "plan", str(d / "in")], capture_output=True, text=True, env=env, check=True)
        return float(r.stdout.split()[0]), r.stdout.split()[1] == "1"

    run.exe, run.env, run.plan = str(exe), env, plan
    return run


def test_stores_cut_differently_have_different_launch_keys(waves):
    assert subprocess.run([waves.exe, "keys"], env=waves.env).returncode == 0


def regular_graph(n, deg, seed):
    idx = np.random.default_rng(seed).integers(0, n, (n, deg))
    return np.arange(n + 1, dtype=np.int64) * deg, np.sort(idx, axis=1).astype(np.int32).ravel()


@pytest.mark.parametrize("B,fan", [(100, [10, 5]), (1000, [15, 10]), (1000, [20, 15, 10]), (4000, [50]), (50, [3, 0, 3])])
def test_expected_edges(waves, B, fan):
    """Within a fifth of what minibatches sample: nodes are taken to be alike inside a
    power of two of degree and in-degree, and a class's sampled nodes to be spread evenly."""
    rng = np.random.default_rng(51)
    n = 20000
    for off, idx in (regular_graph(n, 24, 52), random_graph(2000, 12, 53, hubs=5, hub_deg=900, multi=True),
                     (None, None)):
        if off is None:                                       # in-degrees and degrees skewed alike
            w = 1.0 / (1.0 + np.arange(n)) ** 0.7
            deg = np.minimum(rng.poisson(20 * n * w / w.sum()), 3000)
            off = np.concatenate([[0], np.cumsum(deg)])
            idx = rng.choice(n, off[-1], p=w / w.sum()).astype(np.int32)
        b, nn = min(B, len(off) - 1), len(off) - 1
        o = oracle.Oracle(off, idx)
        real = np.mean([sum(c.size for c in o.minibatch(t, fan, 3, j).col)
                        for j, t in enumerate(np.stack([rng.permutation(nn)[:b] for _ in range(4)]).astype(np.int32))])
        assert abs(waves.plan(off, idx, 1, b, fan)[0] - real) <= 0.2 * real


def test_few_large_minibatches_are_left_to_the_radix_path(waves):
    """One workgroup per range walks its share of a minibatch's edges alone."""
    off, idx = regular_graph(1 << 16, 40, 54)
    use = lambda *a: waves.plan(off, idx, *a)[1]              # noqa: E731
    assert not use(1, 4096, [20, 15, 10]) and not use(2, 4096, [50, 50]) and not use(1, 4096, [25, 20])
    assert use(16, 4096, [20, 15, 10]) and use(1, 256, [15, 10]) and use(8, 1024, [10, 5])
    assert use(1, 700, [39, 39]) and not use(1, 700, [40, 40])    # its sampler is slow above 32 draws of more neighbours


def check(waves, off, idx, targets, fan, bounds, seed=3, mb=2, rpb=16, e_blk_log2=5):
    ref = oracle.Oracle(off, idx).hyperbatch(targets, fan, seed, mb)
    H, L = len(ref), len(fan)
    nodes = np.concatenate([m.nodes for m in ref])
    key = np.concatenate([m.nodes.astype(np.uint64) << np.uint64(32) | np.uint64(j) for j, m in enumerate(ref)])
    order = np.argsort(key, kind="stable")
    val = np.concatenate([np.arange(len(m.nodes), dtype=np.int32) for m in ref])
    want = oracle.hyperbatch_stats(off, 4 << e_blk_log2, (4 << e_blk_log2) // rpb, ref, L)
    for highest_first in (0, 1):
        got = waves(off, idx, targets, fan, bounds, seed, mb, highest_first, rpb, e_blk_log2)
        tag = ("highest first" if highest_first else "lowest first",)
        assert not got["err"].any(), tag
        assert np.array_equal(got["sizes"], np.stack([m.layer_sizes for m in ref])), tag
        assert np.array_equal(got["nodes"], nodes), tag
        for l in range(L):
            assert np.array_equal(got["row_ptr"][l], np.concatenate([m.row_ptr[l] for m in ref])), tag + (l,)
            assert np.array_equal(got["col"][l], np.concatenate([m.col[l] for m in ref])), tag + (l,)
        assert np.array_equal(got["list_key"], key[order]), tag
        assert np.array_equal(got["list_val"], val[order]), tag
        assert got["stats"].tolist() == [want["distinct_rows"], want["feat_blocks"], *want["topo_blocks"]], tag


def test_ranges_without_new_nodes(waves):
    """Between hops, ranges whose sampled neighbours the minibatch already holds, or
    that it does not reach, beside ranges with new nodes."""
    n = 640
    off, idx = random_graph(n, 5, 41, hubs=0)
    held = np.arange(128, 384, dtype=np.int32)                # ranges 1 and 2 are held whole
    t = np.stack([np.random.default_rng(j).permutation(held) for j in range(2)])
    check(waves, off, idx, t, [4, 3], [0, 128, 256, 384, 512, 640])
    off, idx = random_graph(200, 4, 42, hubs=0)               # no edges into the upper ranges
    off = np.concatenate([off, np.full(n - 200, off[-1])])
    check(waves, off, idx, distinct_targets(200, 3, 20, 43), [3, 2, 2], [0, 64, 256, 320, 448, 640])


@pytest.mark.parametrize("fan", [[6, 4], [40, 2], [70], [0, 3], [1, 2, 2, 1]])
def test_hops(waves, fan):
    off, idx = random_graph(900, 9, 44, hubs=3, hub_deg=300, multi=True)
    check(waves, off, idx, distinct_targets(900, 3, 30, 45), fan, [0, 256, 512, 900])


@pytest.mark.parametrize("H,B", [(1, 1), (33, 5), (65, 3), (2, 300)])
def test_minibatches_and_targets(waves, H, B):
    off, idx = random_graph(1100, 6, 46, hubs=2)
    check(waves, off, idx, distinct_targets(1100, H, B, 47), [5, 2], [0, 384, 1100])


def test_bad_targets_are_reported(waves):
    off, idx = random_graph(300, 4, 48)
    t = distinct_targets(300, 4, 6, 49)
    t[1, 3], t[2, 5], t[3, 0] = t[1, 0], 300, -1
    for highest_first in (0, 1):
        got = waves(off, idx, t, [3, 2], [0, 128, 300], 1, 0, highest_first)
        assert got["err"].tolist() == [0, 2, 1, 1]
        assert got["sizes"][1:].max() == 0 and got["sizes"][0, 0] == 6


@pytest.mark.parametrize("n,B,fan,bounds", [
    (9000, 400, [12, 8], [0, 9000]),                          # new and held nodes of one range in several rounds
    (5000, 1100, [1024, 2], [0, 1024, 5000]),                 # chunks of four rows: more than one round locates
    (140000, 30, [5, 3], [0, 256, 140000]),                   # a range of more than 2^17 nodes: 512 threads
])
def test_beyond_one_round(waves, n, B, fan, bounds):
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 25, n) if n < 10000 else rng.integers(0, 9, n)
    off = np.concatenate([[0], np.cumsum(deg)])
    idx = rng.integers(0, n, off[-1]).astype(np.int32)
    t = distinct_targets(n, 1, B, 50)
    if n == 9000:
        m = oracle.Oracle(off, idx).minibatch(t[0], fan, 3, 2)
        assert (np.diff(m.layer_sizes) > 2048).all()          # kNewCap
        assert m.layer_sizes[1] > 512                         # kOldCap
    check(waves, off, idx, t, fan, bounds)
