"""What this framework's speed is measured on.

Each case is work that a program using the framework has it do, through the
package's public entry points (Store, Batch):

  prepare   one hyperbatch, synchronously: sampling, relabelled CSR blocks and
            gathered feature rows (what a training step or a request waits for)
  pipeline  consecutive hyperbatches with begin / finish / wait, the sampling of
            three of them ahead of the gather (a training epoch's data loader)
  staged    consecutive prepares on a store whose features stay in pinned host
            memory, with a pool of feature blocks and a cache of hot rows in HBM
  sage      the GraphSAGE forward over a hyperbatch that is already prepared
  infer     prepare and forward, one inference step

Graphs are R-MAT with distinct edges and no self-loops, features N(0, 1),
targets uniform and distinct within a minibatch.  A data set depends on the case
alone (a program loads it once and keeps its store).  How many nodes and edges a
hyperbatch samples depends on its minibatches' target sets and the sampling seed,
so these are the case's too, and every seed's outputs have the same shapes; the
seed gives the order in which each minibatch lists its targets (and with it the
rows, ids and columns that belong to them) and the model's weights.
"""
import collections
import ctypes
import json
import math

import numpy as np
import torch

import paper_2601_01473_amd as ag

_UNIFORM, _SKEWED = "0.57,0.19,0.19", "0.65,0.15,0.15"


def listed():
    return [
        # one small minibatch at a time: an online request, or data preparation
        # without hyperbatches; all latency and launches
        _prepare("prepare 2^14 1x256", 1 << 14, 16, "float32", 64, 4096, 1, 256, "10,5", offsets="int32"),
        # the smallest hyperbatch workload (8 minibatches on a 2^14-node graph)
        _prepare("prepare 2^14 8x256", 1 << 14, 16, "float32", 64, 4096, 8, 256, "10,5", offsets="int32"),
        # the middle workload: 512-byte rows, int64 offsets, targets on the device
        _prepare("prepare 2^20 32x1024", 1 << 20, 20, "float32", 128, 4096, 32, 1024, "15,10", targets="device"),
        # odd sizes throughout: rows that are no multiple of 16 bytes, a node count
        # and a hyperbatch that are no powers of two, a fanout above 32
        _prepare("prepare 300007 13x777", 300007, 12, "float32", 75, 8192, 13, 777, "7,40", offsets="int32"),
        # skewed degrees and wide rows: 2 KiB bf16 features, 8 minibatches
        _prepare("prepare skew 2^21 8x1024", 1 << 21, 30, "bfloat16", 1024, 4096, 8, 1024, "25,10", abc=_SKEWED),
        # the default workload, one hyperbatch at a time, targets in host memory
        _prepare("prepare 2^23 64x1024", 1 << 23, 30, "float32", 256, 65536, 64, 1024, "25,10"),
        # three hops over a large graph, 256-byte fp16 rows: the largest sampling
        _prepare("prepare 2^24 3-hop 64x1024", 1 << 24, 16, "float16", 128, 65536, 64, 1024, "15,10,5"),
        # an epoch's data loader on the middle and on the default workload
        _prepare("pipeline 2^20 8 x 32x1024", 1 << 20, 20, "float32", 128, 4096, 32, 1024, "15,10", targets="device",
                 kind="pipeline", steps=8),
        _prepare("pipeline 2^23 6 x 64x1024", 1 << 23, 30, "float32", 256, 65536, 64, 1024, "25,10",
                 targets="device", kind="pipeline", steps=6),
        # features larger than the HBM given to them: consecutive hyperbatches,
        # whose blocks together are more than the pool holds
        _prepare("staged 2^20 4 x 16x1024", 1 << 20, 20, "bfloat16", 256, 4096, 16, 1024, "10,5", kind="staged",
                 steps=4, pool=1 << 15, cache=1 << 14),
        # the model step of training or inference on the default workload
        _prepare("sage 2^23 64x1024", 1 << 23, 30, "float32", 256, 65536, 64, 1024, "25,10", kind="sage",
                 dims="256,256"),
        # one inference step on a small hyperbatch, three layers, bf16 features,
        # widths that are no multiples of the GEMM's tile
        _prepare("infer 2^17 8x512 3-layer", 1 << 17, 16, "bfloat16", 96, 4096, 8, 512, "10,5,5", kind="infer",
                 dims="160,160,64"),
    ]


def draw(rng):
    """One more case of the listed ones' ranges: 2^11 to 2^22 nodes, rows of 4 bytes to 4 KiB, 1 to 3 hops with
    fanouts 1 to 50, 1 to 64 minibatches of 16 to 1024 targets."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["prepare"] * 5 + ["pipeline"] * 2 + ["staged", "sage", "sage", "infer"])
    while True:
        dtype = rng.choice(["float32", "float32", "float16", "bfloat16"])
        if kind in ("sage", "infer"):
            dim = 32 * spread(1, 16)
        else:
            dim = spread(1, 1024) if dtype == "float32" else 2 * spread(1, 1024)
        nodes = spread(1 << 11, 1 << 22)
        if rng.random() < 0.3:
            nodes = 1 << (nodes.bit_length() - 1)
        hops = rng.choice([1, 2, 2, 2, 3, 3])
        fan = [rng.choice([5, 10, 15, 20, 25, spread(1, 32), spread(1, 50)]) for _ in range(hops)]
        H, B = spread(1, 64), spread(16, 1024)
        steps = rng.randint(3, 6) if kind == "pipeline" else rng.randint(2, 4) if kind == "staged" else 1
        row = dim * (4 if dtype == "float32" else 2)
        bound = H * min(B * math.prod(1 + f for f in fan), nodes) * steps
        host = kind == "staged" and bound * row > 1 << 29
        if B <= nodes // 2 and nodes * row <= 1 << 31 and bound <= 12 << 20 and bound * row <= 4 << 30 and not host:
            break
    block = 1 << rng.randint(max(12, (row - 1).bit_length()), 17)
    blocks = -(-nodes // (block // row))
    case = _prepare("", nodes, rng.choice([4, 8, 16, 20, 30]), dtype, dim, block, H, B, ",".join(map(str, fan)),
                    offsets=rng.choice(["int32", "int64"]), targets=rng.choice(["host", "device"]),
                    abc=rng.choice([_UNIFORM, _UNIFORM, _SKEWED]), kind=kind, steps=steps)
    if kind == "staged":
        case["pool"] = max(1, int(blocks * rng.uniform(0.1, 0.9)))
        case["cache"] = rng.choice([0, max(1, int(nodes * rng.uniform(0.01, 0.2)))])
    if kind in ("sage", "infer"):
        case["dims"] = ",".join(str(32 * spread(1, 16)) for _ in range(hops))
    del case["name"]
    return case


def _prepare(name, nodes, degree, dtype, dim, block, H, B, fanouts, offsets="int64", targets="host", abc=_UNIFORM,
             kind="prepare", steps=1, **more):
    return dict(name=name, kind=kind, nodes=nodes, degree=degree, abc=abc, offsets=offsets, dtype=dtype, dim=dim,
                block=block, H=H, B=B, fanouts=fanouts, targets=targets, steps=steps, **more)


# ----------------------------------------------------------------- data sets

def _graph(n, degree, abc, gen):
    """R-MAT edges (ids not permuted) as CSR in host memory: offsets int64 [n + 1], indices int32."""
    a, b, c = (float(x) for x in abc.split(","))
    left, keys = n * degree, []
    while left > 0:
        m = min(left, 1 << 25)
        left -= m
        src = torch.zeros(m, dtype=torch.int64, device="cuda")
        dst = torch.zeros_like(src)
        for _ in range(max(1, (n - 1).bit_length())):
            r = torch.rand(m, device="cuda", generator=gen)
            src = 2 * src + (r >= a + b)
            dst = 2 * dst + (((r >= a) & (r < a + b)) | (r >= a + b + c))
        keep = (src < n) & (dst < n) & (src != dst)
        keys.append((src * n + dst)[keep])
    key = torch.cat(keys).sort().values
    del keys
    key = key[torch.cat([key.new_ones(1, dtype=torch.bool), key[1:] != key[:-1]])]
    src = torch.div(key, n, rounding_mode="floor")
    off = torch.searchsorted(src, torch.arange(n + 1, device="cuda"))
    return off.cpu().numpy(), (key - src * n).to(torch.int32).cpu().numpy()


def _features(n, dim, dtype, gen):
    out = np.empty((n, dim), dtype={"float32": np.float32, "float16": np.float16, "bfloat16": np.uint16}[dtype])
    host = torch.from_numpy(out.view(np.int16) if dtype == "bfloat16" else out)
    rows = max(1, (1 << 27) // dim)
    for i in range(0, n, rows):
        x = torch.randn(min(rows, n - i), dim, device="cuda", generator=gen).to(getattr(torch, dtype))
        host[i:i + rows].copy_(x.view(torch.int16) if dtype == "bfloat16" else x)
    return out


_stores = collections.OrderedDict()     # a few data sets at a time, as a program keeps the one it works on


def _store(case):
    parts = [case[k] for k in ("nodes", "degree", "abc", "offsets", "dtype", "dim", "block")]
    tier = dict(pool_blocks=case["pool"], cache_rows=case["cache"] or None) if case["kind"] == "staged" else {}
    key = json.dumps([parts, tier])
    if key not in _stores:
        while len(_stores) >= 2:
            _stores.popitem(last=False)
        gen = torch.Generator(device="cuda").manual_seed(case["nodes"] * 31 + case["degree"])
        off, idx = _graph(case["nodes"], case["degree"], case["abc"], gen)
        feat = _features(case["nodes"], case["dim"], case["dtype"], gen)
        torch.cuda.empty_cache()
        _stores[key] = ag.Store(off.astype(case["offsets"]), idx, feat, case["block"], feat_dtype=case["dtype"], **tier)
    _stores.move_to_end(key)
    return _stores[key]


# ----------------------------------------------------------------- states

class _Memory:
    """A batch's device array; keeps the batch, and so the memory, while a tensor on it lives."""

    def __init__(self, batch, ptr, n, kind):
        self.batch = batch
        self.__cuda_array_interface__ = dict(data=(ptr, False), shape=(n,), typestr=kind, version=2)


def _tensor(batch, ptr, n, kind):
    if not n:
        return torch.empty(0, dtype=getattr(torch, {"<i4": "int32", "<f4": "float32", "<f2": "float16",
                                                    "<i2": "int16"}[kind]), device="cuda")
    return torch.as_tensor(_Memory(batch, ptr, n, kind), device="cuda")


class _Sizes(np.ndarray):
    """layer_sizes in the library's memory; keeps the batch too."""


class _Arrays:
    """A prepared batch's arrays as tensors on its own buffers; made again only when a buffer or a size has changed."""

    def __init__(self, dtype):
        self.dtype, self.key, self.out = dtype, None, None

    def __call__(self, batch):
        v = batch.view()
        H, L = v.H, v.L
        rows = v.node_off[H]
        key = [v.nodes, v.features, rows, ctypes.addressof(v.layer_sizes.contents)]
        for l in range(L):
            key += [v.row_ptr[l], v.rp_off[l][H], v.col[l], v.col_off[l][H]]
        if key != self.key:
            kind = {"float32": "<f4", "float16": "<f2", "bfloat16": "<i2"}[self.dtype]
            width = v.row_bytes // int(kind[2])
            feat = _tensor(batch, v.features, rows * width, kind)
            feat = feat.view(torch.bfloat16) if self.dtype == "bfloat16" else feat
            sizes = np.frombuffer((ctypes.c_int32 * (H * (L + 1))).from_address(key[3]), np.int32)
            sizes = sizes.reshape(H, L + 1).view(_Sizes)
            sizes.batch = batch
            self.out = dict(nodes=_tensor(batch, v.nodes, rows, "<i4"), features=feat.view(rows, width),
                            layer_sizes=sizes,
                            row_ptr=[_tensor(batch, v.row_ptr[l], v.rp_off[l][H], "<i4") for l in range(L)],
                            col=[_tensor(batch, v.col[l], v.col_off[l][H], "<i4") for l in range(L)])
            self.key = key
        return self.out


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.kind, s.store, s.H, s.steps = case["kind"], _store(case), case["H"], case["steps"]
    s.fanouts = [int(f) for f in case["fanouts"].split(",")]
    n, B = case["nodes"], case["B"]
    s.seed, s.mb = n + s.H, 5 * s.H
    sets, order = np.random.default_rng(n + B), np.random.default_rng(int(seed))
    s.targets = []
    for _ in range(s.steps):
        if s.H * B <= n:
            t = sets.choice(n, s.H * B, replace=False).reshape(s.H, B)
        else:
            t = np.stack([sets.choice(n, B, replace=False) for _ in range(s.H)])
        t = np.ascontiguousarray(order.permuted(t, axis=1), dtype=np.int32)
        s.targets.append(torch.from_numpy(t).cuda() if case["targets"] == "device" else t)
    s.batches = [None] * s.steps
    s.arrays = [_Arrays(case["dtype"]) for _ in range(s.steps)]
    if s.kind == "pipeline":
        s.streams = [torch.cuda.Stream() for _ in range(3)]
    if s.kind in ("sage", "infer"):
        gen = torch.Generator(device="cuda").manual_seed(int(seed))
        dims = [case["dim"]] + [int(d) for d in case["dims"].split(",")]
        s.weights = [(torch.randn(o, 2 * i, device="cuda", generator=gen) / math.sqrt(2 * i)).bfloat16()
                     for i, o in zip(dims, dims[1:])]
        s.biases = [0.1 * torch.randn(o, device="cuda", generator=gen) for o in dims[1:]]
        s.out = torch.empty(s.H * B, dims[-1], device="cuda")
    if s.kind == "sage":
        _one(s)
    return s


def _one(s, i=0):
    s.batches[i] = s.store.prepare(s.targets[i], s.fanouts, seed=s.seed, mb_base=s.mb + i * s.H, batch=s.batches[i])
    return s.batches[i]


def run(s):
    if s.kind == "sage":
        return s.batches[0].sage_forward(s.weights, s.biases, out=s.out)
    if s.kind == "infer":
        logits = _one(s).sage_forward(s.weights, s.biases, out=s.out)
        return dict(batch=s.arrays[0](s.batches[0]), logits=logits)
    if s.kind != "pipeline":
        return [s.arrays[i](_one(s, i)) for i in range(s.steps)]
    ahead = 3

    def begin(i):
        s.batches[i] = s.store.begin(s.targets[i], s.fanouts, seed=s.seed, mb_base=s.mb + i * s.H, batch=s.batches[i],
                                     stream=s.streams[i % len(s.streams)])

    for i in range(min(ahead, s.steps)):
        begin(i)
    for i in range(s.steps):
        s.batches[i].finish()
        if i + ahead < s.steps:
            begin(i + ahead)
    return [a(b.wait()) for a, b in zip(s.arrays, s.batches)]


# ----------------------------------------------------------------- what is measured against

def work(case):
    """Counts of one hyperbatch of these sizes.  Sampling: per request its id, two offsets and its row pointer; per
    sampled edge the index read and the column written; per new node its id.  Gather: the distinct rows read and every
    minibatch's rows and ids written.  Forward: rows, CSR, weights and biases read, embeddings written; the GEMMs."""
    s = prepare(dict(case, kind="staged" if case["kind"] == "staged" else "prepare", steps=1), 1)
    st = _one(s).stats()
    size = 4 if case["dtype"] == "float32" else 2
    row = case["dim"] * size
    data = sum(16 * r + 8 * e + 4 * u for r, e, u in zip(st["requests"], st["sampled"], st["new_nodes"]))
    data += st["rows"] * (4 + row) + st["distinct_rows"] * row
    if "dims" not in case:
        return dict(bytes=data * case["steps"], flops=0)
    dims = [case["dim"]] + [int(d) for d in case["dims"].split(",")]
    forward = st["rows"] * row + sum(4 * (r + case["H"] + e) for r, e in zip(st["requests"], st["sampled"]))
    forward += sum(4 * i * o + 4 * o for i, o in zip(dims, dims[1:])) + 4 * case["H"] * case["B"] * dims[-1]
    flops = sum(4 * m * i * o for m, i, o in zip(reversed(st["requests"]), dims, dims[1:]))
    return dict(bytes=forward + (data if case["kind"] == "infer" else 0), flops=flops)


def tolerance(case):
    """Ids, row pointers, columns and feature rows are whole values and copies.  The forward rounds its operands and
    hidden embeddings to bf16: measured 2e-3 to 2.6e-3 off the 64-bit result for one to three layers."""
    return {"rel": 1e-2, "max": 0.1} if "dims" in case else "exact"


def exact(case, seed):
    """The forward in 64 bits over the prepared hyperbatch's own CSR blocks and rows, from the bf16 weights as given."""
    if "dims" not in case:
        return None
    s = prepare(case, seed)
    a = s.arrays[0](s.batches[0] or _one(s))
    sizes, L = np.array(a["layer_sizes"], dtype=np.int64), len(s.fanouts)
    start = np.concatenate([[0], np.cumsum(sizes[:, L])])
    h = a["features"]
    for i in range(L):
        hop = L - 1 - i
        w, b = s.weights[i].double(), s.biases[i].double()
        out, rp, e = [], 0, 0
        for j in range(s.H):
            m = int(sizes[j, hop])
            x = h[int(start[j]):int(start[j + 1])]
            ptr = a["row_ptr"][hop][rp:rp + m + 1].long()
            deg = ptr[1:] - ptr[:-1]
            col = a["col"][hop][e:e + int(ptr[-1])].long()
            rp, e = rp + m + 1, e + len(col)
            mean = torch.zeros(m, x.shape[1], dtype=torch.float64, device="cuda")
            mean.index_add_(0, torch.repeat_interleave(torch.arange(m, device="cuda"), deg), x[col].double())
            mean /= deg.clamp(min=1).double()[:, None]
            z = torch.cat([x[:m].double(), mean], 1) @ w.T + b
            out.append(z.relu() if i + 1 < L else z)
        h = torch.cat(out)
        start = np.concatenate([[0], np.cumsum(sizes[:, hop])])
    return h if case["kind"] == "sage" else dict(batch=None, logits=h)
