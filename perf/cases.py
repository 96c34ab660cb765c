"""What a user of this package has it do, as measurable cases: training steps, evaluation and message encoding on
graphs of the package's own configurations and of sizes between and around them.

A case's graph, node-to-partition map and index structures are fixed by the case (a training program loads its graph
once and keeps it); features, weights, upstream gradients, labels and the mask key come from the seed. Every pass of a
training case is one step further: the kept positions of the exchange change from pass to pass.

Kinds of a case
  step     gradients cleared, forward and backward of the whole network, upstream gradient given
  train    one iteration of Algorithm 1: forward, loss, backward, summed weight gradients, gradient step
  replay   the step captured once in a HIP graph and replayed
  eval     forward and loss on the held-out nodes, nothing kept for a backward pass
  ktap     step of a network whose layers have more than two taps
  codec    encoder, decoder and owner-side decoder-with-sum on boundary rows, as separate calls
"""
import math
from collections import OrderedDict

import numpy as np
import torch

from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import KTapNetwork, PartitionedNetwork

_MEDIUM = dict(graph="power", nodes=169_343, edges=1_166_243, exponent=2.5)
_LARGE = dict(graph="power", nodes=2_449_029, edges=61_859_140, exponent=2.3)


def _case(name, kind, widths, ratio, conv="gcn", parts=4, cut="random", dtype="f32", streams=1, first=-1, taps=2, **graph):
    c = dict(kind=kind, widths=widths, ratio=ratio, conv=conv, parts=parts, cut=cut, dtype=dtype, streams=streams,
             transform_first=first, taps=taps, **graph)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration, where a step is nothing but launches and host work
        _case("tiny_step", "step", "16-32-8", "4/1", parts=2, cut="blocks", graph="sbm", nodes=2000, edges=0, exponent=0.0),
        # the training demo: eight partitions of a block-model graph, every call of an iteration
        _case("demo_train", "train", "32-64-8", "4/1", conv="sage", parts=8, graph="sbm_demo", nodes=16000, edges=0, exponent=0.0),
        # the citation-sized graph at a usual ratio, as bench.py runs it (two streams)
        _case("medium_step", "step", "128-256-256-40", "8/1", streams=2, **_MEDIUM),
        # the same network trained with full communication (the start of every comparison, the end of every schedule)
        _case("medium_full_train", "train", "128-256-256-40", "1/1", **_MEDIUM),
        # sixteen low-cut partitions at the middle of the 16 -> 1 schedule, replayed from a HIP graph
        _case("medium_bfs16_replay", "replay", "128-256-256-40", "834/99", parts=16, cut="bfs", **_MEDIUM),
        # nothing a power of two: odd node count, five partitions, widths with remainders, an odd ratio
        _case("ragged_step", "step", "75-200-136-47", "3/1", conv="sage", parts=5, graph="power", nodes=50_021, edges=500_009,
              exponent=2.4),
        # evaluation of held-out nodes on a graph between the two datasets
        _case("eval_forward", "eval", "100-256-256-47", "2/1", conv="sage", parts=8, graph="power", nodes=410_003,
              edges=6_150_001, exponent=2.3),
        # general layers of eq. (1): two hops of exchange per layer
        _case("ktap3_step", "ktap", "64-128-24", "4/1", conv="sage", parts=3, taps=3, graph="power", nodes=60_013, edges=480_007,
              exponent=2.5),
        # bf16 storage, few partitions, the class layer transforming before it aggregates
        _case("class_first_bf16", "step", "128-512-512-40", "4/1", dtype="bf16", first=2, streams=2, **_MEDIUM),
        # the encoder and both decoders as calls of their own, rows of a hidden layer
        _case("codec_f32", "codec", "256-8", "8/1", graph="rows", nodes=600_011, edges=450_007, exponent=0.0, parts=1),
        # the two large configurations, as bench.py runs them
        _case("large_sage_step", "step", "100-256-256-47", "8/1", conv="sage", parts=8, streams=2, **_LARGE),
        _case("large_gcn_bf16_step", "step", "100-512-512-47", "4/1", parts=32, dtype="bf16", streams=2, **_LARGE),
    ]


_MOST = None


def draw(rng):
    """One more case of the same ranges: graphs of 2,000 to 1.2 million nodes, 4 to 60 neighbours, 2 to 32 partitions,
    inputs of 16 to 256 features (odd widths included), hidden widths of 32 to 512, 5 to 64 classes, ratios of 1 to 32."""
    global _MOST
    if _MOST is None:
        _MOST = max(_cost(c) for c in listed())
    log_uniform = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    while True:
        kind = rng.choice(["step", "step", "step", "train", "train", "replay", "eval", "ktap", "codec"])
        dtype = rng.choice(["f32", "f32", "bf16"])
        ratio = rng.choice(["1/1", "2/1", "3/1", "4/1", "8/1", "16/1", "32/1", "834/99", "7/2", "1/0"])
        nodes = log_uniform(2_000, 1_200_000)
        if kind == "codec":
            width = 4 * rng.randint(4, 128) if rng.random() < 0.75 else rng.randint(16, 512)
            ratio = "8/1" if ratio == "1/0" else ratio
            c = _case(None, kind, "%d-8" % width, ratio, dtype=dtype, graph="rows", nodes=nodes,
                      edges=max(1, int(nodes * rng.uniform(0.3, 1.0))), exponent=0.0, parts=1)
        else:
            edges = int(nodes * math.exp(rng.uniform(math.log(2.0), math.log(30.0))))
            conv = "sage" if kind == "ktap" else rng.choice(["gcn", "sage"])
            hidden = [8 * log_uniform(4, 64) for _ in range(2 if kind != "ktap" and rng.random() < 0.6 else 1)]
            widths = [rng.randint(16, 256)] + hidden + [rng.randint(5, 64)]
            first = -1
            if dtype == "bf16" and kind in ("step", "train") and widths[-2] % 16 == 0 and rng.random() < 0.3:
                first = len(widths) - 2
            parts = log_uniform(2, 32) if kind != "ktap" else log_uniform(2, 8)
            c = _case(None, kind, "-".join(map(str, widths)), ratio, conv=conv, parts=parts, dtype=dtype,
                      streams=1 if kind == "ktap" or parts == 2 else rng.choice([1, 2]), first=first,
                      taps=rng.choice([3, 4]) if kind == "ktap" else 2, graph="power", nodes=nodes, edges=edges,
                      exponent=round(rng.uniform(2.2, 2.8), 2))
        if _cost(c) <= 0.5 * _MOST:
            return c


# ---------------------------------------------------------------------------------------------------------------
# what a user's program has in hand: graph, partitions, network, inputs
# ---------------------------------------------------------------------------------------------------------------

_structures = OrderedDict()      # the last few graphs of this process, partitioned
_KEEP = 6


def _structure(c):
    """Index structures of every partition (the host-side builder's arrays)."""
    key = tuple(c[k] for k in ("graph", "nodes", "edges", "exponent", "conv", "cut", "parts"))
    if key in _structures:
        _structures.move_to_end(key)
        return _structures[key]
    operator = synth.gcn_operator if c["conv"] == "gcn" else synth.sage_mean_operator
    n = c["nodes"]
    if c["graph"] == "sbm":
        half = n // 2
        g = operator(*synth.sbm_edges((half, n - half), 0.01, 0.0005, synth.SEED_GRAPH))
    elif c["graph"] == "sbm_demo":
        size = n // 8
        g = operator(*synth.sbm_edges((size,) * 8, 8.0 / size, 1.0 / size, synth.SEED_GRAPH + 100))
    else:
        g = operator(n, *synth.chung_lu_edges(n, c["edges"], c["exponent"], synth.SEED_GRAPH))
    if c["cut"] == "blocks":
        part = synth.block_partition((n // 2, n - n // 2))
    elif c["cut"] == "bfs":
        part = synth.bfs_contiguous_partition(g, c["parts"])
    else:
        part = synth.random_partition(n, c["parts"], synth.SEED_PART)
    host = vb.partition_build(n, g.rowptr, g.colidx, g.vals, part, c["parts"])
    while len(_structures) >= _KEEP:
        _structures.popitem(last=False)
    _structures[key] = host
    return host


def _widths(c):
    return tuple(int(w) for w in c["widths"].split("-"))


def _ratio(c):
    num, den = c["ratio"].split("/")
    return int(num), int(den)


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    s.kind, s.ratio, s.step = c["kind"], _ratio(c), 0
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    host_rng = np.random.default_rng(seed)
    key = int(host_rng.integers(1, 1 << 62))
    widths = _widths(c)
    if s.kind == "codec":
        return _prepare_codec(c, s, widths, key, gen, host_rng)
    host = _structure(c)
    n, L = c["nodes"], len(widths) - 1
    if s.kind == "ktap":
        net = KTapNetwork(host, widths, c["taps"], key, dtype=c["dtype"])
        net.set_tap_weights([[_glorot(host_rng, widths[l], widths[l + 1]) for _ in range(c["taps"])] for l in range(L)])
    else:
        first = (c["transform_first"],) if c["transform_first"] >= 0 else ()
        net = PartitionedNetwork(host, widths, c["conv"], key, need_backward=s.kind != "eval", dtype=c["dtype"],
                                 n_streams=c["streams"], transform_first=first)
        net.set_weights([_glorot(host_rng, widths[l], widths[l + 1]) for l in range(L)],
                        [_glorot(host_rng, widths[l], widths[l + 1]) for l in range(L)])
    net.x[0].copy_(torch.randn(n, widths[0], generator=gen, device="cuda"))
    if s.kind in ("train", "eval"):
        net.set_labels(host_rng.integers(0, widths[-1], n, dtype=np.int32), host_rng.random(n) < 0.5)
    else:
        net.dx[L].copy_(torch.randn(n, widths[-1], generator=gen, device="cuda") / n)
    s.net, s.L = net, L
    if s.kind == "replay":
        s.graph = net.capture_step(s.ratio)
    return s


def _glorot(rng, fan_in, fan_out):
    lim = math.sqrt(6.0 / (fan_in + fan_out))
    return ((rng.random((fan_in, fan_out), dtype=np.float32) * 2.0 - 1.0) * lim).astype(np.float32)


def _prepare_codec(c, s, widths, key, gen, host_rng):
    # `edges` of the `nodes` rows of a partition are boundary rows, ascending; node ids of a larger graph
    n, b, width = c["nodes"], c["edges"], widths[0]
    bf16 = c["dtype"] == "bf16"
    s.ctx = vb.Context(list(widths), [vb.ACT_RELU], vb.CONV_GCN, 1, key, vb.BF16 if bf16 else vb.F32)
    s.ctx.prepare()
    s.ctx.set_ratio(-1, *s.ratio)
    dt = torch.bfloat16 if bf16 else torch.float32
    s.rows = torch.randperm(n, generator=gen, device="cuda")[:b].sort().values.to(torch.int32)
    s.gids = (s.rows * 3 + 1).to(torch.int32)
    s.x = torch.randn(n, width, generator=gen, device="cuda").to(dt)
    s.grad = torch.randn(n, width, generator=gen, device="cuda").to(dt)
    s.z = torch.empty(b * s.ctx.keep(0), dtype=dt, device="cuda")
    s.dense = torch.empty(b, width, dtype=dt, device="cuda")
    s.n_rows, s.width = b, width
    return s


_LEARNING_RATE = 0.01


def run(state):
    s = state
    s.step += 1
    if s.kind == "codec":
        s.ctx.begin_step(s.step)
        s.ctx.compress(0, s.gids, s.rows, s.n_rows, s.x, s.width, s.z)
        s.ctx.decompress(0, s.gids, None, s.n_rows, s.z, s.dense, s.width, False)
        s.ctx.decompress(0, s.gids, s.rows, s.n_rows, s.z, s.grad, s.width, True)
        return {"z": s.z, "dense": s.dense, "grad": s.grad}
    net = s.net
    if s.kind == "train":
        totals = net.train_step(s.step, s.ratio, _LEARNING_RATE)
        return {"totals": totals, "logits": net.x[s.L], "h1": net.h1, "h0": net.h0, "dh1": net.dh1, "dh0": net.dh0,
                "dx": net.dx[1:s.L]}
    if s.kind == "eval":
        net.forward(s.step, s.ratio)
        return {"totals": net.loss(train=False, with_gradient=False), "logits": net.x[s.L]}
    net.zero_grads()
    if s.kind == "replay":
        s.graph.replay()
    else:
        net.step(s.step, s.ratio)
    if s.kind == "ktap":
        return {"logits": net.x[s.L], "dh": net.dh, "dx": net.dx[1:s.L]}
    return {"logits": net.x[s.L], "dh1": net.dh1, "dh0": net.dh0, "dx": net.dx[1:s.L]}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------

def _counts(c):
    """(stored entries, halo rows over all partitions, boundary rows, share of halo entries)."""
    n, parts = c["nodes"], c["parts"]
    if c["graph"] in ("sbm", "sbm_demo") or c["cut"] != "random":
        host = _structure(c)
        nnz = sum(h.nnz for h in host)
        local = sum(int(h.t_rowptr[h.n_local]) for h in host)
        return nnz, sum(h.n_halo for h in host), sum(h.n_boundary for h in host), 1.0 - local / max(1, nnz)
    # expected degrees of the power-law graph; a node with d neighbours reaches (P - 1)(1 - (1 - 1/P)^d) other partitions
    w = (np.arange(n, dtype=np.float64) + 1.0) ** (-1.0 / (c["exponent"] - 1.0))
    for _ in range(8):
        w *= (2.0 * c["edges"]) / w.sum()
        np.minimum(w, math.sqrt(2.0 * c["edges"]), out=w)
    own = n if c["conv"] == "gcn" else 0
    nnz = 2 * c["edges"] + own
    halo = (parts - 1) * float((1.0 - (1.0 - 1.0 / parts) ** w).sum())
    boundary = float((1.0 - (1.0 / parts) ** w).sum())
    return nnz, halo, boundary, 2 * c["edges"] * (1.0 - 1.0 / parts) / nnz


def _keep(width, ratio):
    num, den = ratio
    return 0 if den == 0 else max(1, -(-width * den // num))


def work(case):
    """Bytes: per layer and direction every stored entry (column and value), every activation, aggregate, message and
    gradient row that a call is given or gives back, once; weights and their gradients once. Flops: the dense products
    and one multiply-add per entry and element that reaches a sum."""
    c = case
    widths, ratio = _widths(c), _ratio(c)
    es = 2 if c["dtype"] == "bf16" else 4
    n, L = c["nodes"], len(widths) - 1
    if c["kind"] == "codec":
        b, w, k = c["edges"], widths[0], _keep(widths[0], ratio)
        # kept elements read and written, dense rows written, kept positions of the gradient rows added to
        return {"bytes": float(b) * ((2 * k) + (k + w) + 3 * k) * es + 8.0 * b, "flops": float(b) * k}
    nnz, halo, boundary, cross = _counts(c)
    hops = c["taps"] - 1 if c["kind"] == "ktap" else 1
    mats = c["taps"] if c["kind"] == "ktap" else (2 if c["conv"] == "sage" else 1)
    backward = c["kind"] != "eval"
    nbytes = flops = 0.0
    for l in range(L):
        fi, fo, k = widths[l], widths[l + 1], _keep(widths[l], ratio)
        gather = nnz * ((1.0 - cross) * fi + cross * k)
        nbytes += hops * (8.0 * nnz + 4.0 * n + (boundary + halo) * k * es + n * fi * es) + n * (fi + fo) * es + 4.0 * mats * fi * fo
        flops += 2.0 * hops * gather + 2.0 * mats * n * fi * fo
        if not backward:
            continue
        nbytes += (n * fi * mats + 2.0 * n * fo) * es + 8.0 * mats * fi * fo          # dH from the saved rows, dX_out and the gate
        flops += 2.0 * mats * n * fi * fo
        if l > 0:
            nbytes += hops * (8.0 * nnz + 4.0 * n + (2.0 * halo + 2.0 * boundary) * k * es) + n * fi * es
            flops += 2.0 * hops * gather + 2.0 * mats * n * fi * fo
    if c["kind"] in ("train", "eval"):
        nbytes += n * widths[-1] * es * (2 if backward else 1) + 12.0 * n
    return {"bytes": nbytes, "flops": flops}


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50.0)


def tolerance(case):
    if case["kind"] == "codec":
        return "exact"               # copies, and one addition per element
    if case["dtype"] == "bf16":      # every stored activation, message and gradient is rounded to 8 bits
        return {"rel": 1e-2, "max": 0.5}
    if case["kind"] == "eval":
        return {"rel": 1e-5}         # chained fp32 sums
    # fp32 sums, but a ReLU gate whose argument is within rounding of zero (about one element in 1e7) may open on one side
    # only: sqrt(1e-7) of a gradient's norm, and the whole of the few elements it feeds
    return {"rel": 1e-3, "max": 0.5}
