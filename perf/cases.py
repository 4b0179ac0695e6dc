"""Performance cases of the mini-batch preparation path and its consumers on one MI355X.

A case is a dict of plain values.  Five kinds of work, each through the package's public calls:

  sample     sample_mfg / sample_mfg_many / sample_mfg_static: blocks, node ids, feature rows (and
             labels) of one batch or of one launch set
  epoch      BatchPipeline with a three-layer GraphSAGE forward as the consumer: part of an epoch
  gather     gather_rows: the slice x[ids] alone
  aggregate  mean_aggregate over one block
  layer      sage_layer over one block

Graphs are directed Chung-Lu graphs with the power laws, sizes and maximum degrees of the package's
workloads: a node of weight p has about num_edges * p neighbours, and is drawn as a neighbour with
probability p.  Everything is made on the GPU from the case and the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2110_08450_amd import binding as smfg
from paper_2110_08450_amd import synth
from paper_2110_08450_amd.pipeline import BatchPipeline

DEV = "cuda:0"
DTYPES = {"f16": torch.float16, "f32": torch.float32, "u8": torch.uint8}
SIZE = {"f16": 2, "f32": 4, "u8": 1}

# graph shapes: nodes, directed edges, degree of the heaviest node, mild second law (citations)
TINY = dict(nodes=10_000, edges=100_000, hub=300, mild=False)
ARXIV = dict(nodes=169_000, edges=2_300_000, hub=13_000, mild=False)
PRODUCTS = dict(nodes=2_450_000, edges=124_000_000, hub=17_000, mild=False)
PAPERS = dict(nodes=111_000_000, edges=3_200_000_000, hub=100_000, mild=True)
# an eighth of the papers100M shape: far beyond every cache as well, and quick to make
CITATIONS = dict(nodes=13_900_000, edges=400_000_000, hub=50_000, mild=True)


def listed():
    return [
        # one small batch at a time, as in a test or on a toy data set: latency and launches
        dict(name="tiny_batch", kind="sample", call="one", **TINY, dim=32, dtype="f32", fanouts="10,5", seeds=256,
             batches=1, labels=False),
        # a prediction request for a handful of nodes, by a server that allocates nothing
        dict(name="request_static", kind="sample", call="static", **PRODUCTS, dim=100, dtype="f16",
             fanouts="15,10,5", seeds=16, batches=1, labels=False),
        # training on an arxiv-sized graph, six batches per launch set, the last one partial, with labels
        dict(name="arxiv_set", kind="sample", call="many", **ARXIV, dim=128, dtype="f32", fanouts="15,10,5", seeds=1024,
             batches=6, labels=True),
        # training on a products-sized graph, one batch per call
        dict(name="products_batch", kind="sample", call="one", **PRODUCTS, dim=100, dtype="f16", fanouts="15,10,5",
             seeds=1024, batches=1, labels=False),
        # training on a papers100M-sized graph, eight batches per launch set
        dict(name="papers_set", kind="sample", call="many", **PAPERS, dim=128, dtype="f16", fanouts="15,10,5", seeds=1024,
             batches=8, labels=False),
        # inference on the same graph with large sampled neighbourhoods, one batch per call
        dict(name="papers_infer", kind="sample", call="one", **PAPERS, dim=128, dtype="f16", fanouts="20,20,20",
             seeds=4096, batches=1, labels=False),
        # inference with fanouts beyond one lane per slot, and with whole neighbourhoods
        dict(name="products_wide", kind="sample", call="many", **PRODUCTS, dim=100, dtype="f16", fanouts="100,100",
             seeds=1024, batches=4, labels=False),
        dict(name="products_all", kind="sample", call="one", **PRODUCTS, dim=100, dtype="f16", fanouts="-1,-1", seeds=256,
             batches=1, labels=False),
        # preparation hidden behind a model that runs on the same GPU
        dict(name="epoch_forward", kind="epoch", **CITATIONS, dim=128, dtype="f16", fanouts="15,10,5", seeds=1024,
             batches=16, per_set=4, hidden=256, classes=172),
        # the slice alone, rows of an odd width
        dict(name="gather_odd", kind="gather", nodes=2_450_000, dim=301, dtype="f16", rows=400_000),
        # consumers of the outermost block of a products- and of a papers100M-sized batch
        dict(name="mean_products", kind="aggregate", dst=96_000, fanout=5, fresh=0.55, dim=100, dtype="f16"),
        dict(name="layer_papers", kind="layer", dst=154_321, fanout=5, fresh=0.94, dim=128, out_dim=256, dtype="f16",
             relu=True),
    ]


# ---- cases drawn from the same ranges ------------------------------------------------------------

def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["sample"] * 6 + ["epoch", "gather", "gather", "aggregate", "layer", "layer"])
    if kind == "gather":
        dtype = rng.choice(["f16", "f16", "f32", "u8"])
        dim = rng.choice([rng.randint(1, 700), 8 * rng.randint(1, 64)])
        row = dim * SIZE[dtype]
        return dict(kind=kind, nodes=_log(rng, 1_000, max(2_000, min(20_000_000, 4_000_000_000 // row))), dim=dim, dtype=dtype,
                    rows=_log(rng, 64, max(128, min(4_000_000, 1_000_000_000 // row))))
    if kind in ("aggregate", "layer"):
        fanout = rng.choice([3, 5, 5, 10, 15, 20, 64])
        c = dict(kind=kind, dst=_log(rng, 200, 1_500_000 // fanout), fanout=fanout, fresh=round(rng.uniform(0.3, 0.95), 3),
                 dim=8 * rng.randint(1, 32), dtype=rng.choice(["f16", "f16", "f32"]))
        if kind == "aggregate":
            c["dim"] = rng.choice([c["dim"], rng.randint(1, 300)])
        else:
            c["out_dim"] = rng.choice([256, rng.randint(1, 300)])
            c["relu"] = rng.random() < 0.7
        return c
    while True:
        nodes = _log(rng, 5_000, 30_000_000)
        edges = int(min(500_000_000, nodes * rng.uniform(8, 60)))
        c = dict(kind=kind, nodes=nodes, edges=edges, hub=max(50, min(nodes // 8, _log(rng, 200, 60_000))),
                 mild=rng.random() < 0.5, dim=rng.choice([32, 100, 128, 128, 200, rng.randint(1, 300)]),
                 dtype=rng.choice(["f16", "f32"]))
        seeds = min(nodes // 64, _log(rng, 1, 4096))
        if kind == "epoch":
            c.update(dim=8 * rng.randint(4, 32), dtype="f16", fanouts=rng.choice(["15,10,5", "10,10,5", "12,7"]),
                     seeds=max(1, min(seeds, 1024)), batches=rng.randint(5, 16), per_set=rng.choice([2, 4, 8]),
                     hidden=rng.choice([64, 128, 256]), classes=rng.randint(2, 200))
        else:
            fan = rng.choice(["15,10,5"] * 3 + ["10,5", "20,20,20", "25,10", "7,3,2,2", "32,3", "40,20", "100,100", "-1,5", "-1"])
            c.update(call="one", fanouts=fan, seeds=max(1, seeds), batches=1, labels=rng.random() < 0.3)
            if rng.random() < 0.5:
                c.update(call="many", batches=rng.randint(2, 6 if fan.count(",") < 3 else 4))
            elif c["seeds"] <= 32 and "-" not in fan:
                c.update(call="static")
        n, e, cap = _sizes(c), _fans(c), 1
        cap = c["seeds"] * math.prod(1 + d for d in e if d > 0) if min(e) > 0 else nodes
        cap = min(cap, nodes)
        total = c["batches"] * (n[0][-1] * c["dim"] * SIZE[c["dtype"]] + 8 * sum(n[1]))
        buffers = c["batches"] * (cap * c["dim"] * SIZE[c["dtype"]] + (24 * edges if min(e) < 0 else 40 * cap))
        if total < 3e9 and buffers < 12e9 and nodes * c["dim"] * SIZE[c["dtype"]] < 12e9:
            return c


# ---- the power laws ------------------------------------------------------------------------------

def _fans(c):
    return [int(d) for d in c["fanouts"].split(",")]


def _laws(c):
    """Exponent, offset and normalisation of the one or two rank laws w_r ~ (r + i0)^-alpha."""
    a_dst = 1.0 / 1.5
    a_src = 1.0 / 2.5 if c["mild"] else a_dst
    n = c["nodes"]
    i0 = synth.solve_i0(n, c["edges"] // 2, a_src, a_dst, float(c["hub"]))
    return i0, [(a, i0 ** (1 - a), (n + i0) ** (1 - a)) for a in ([a_src, a_dst] if c["mild"] else [a_dst])]


def _prob(r, i0, laws):
    """Probability of the node of rank r (numpy or torch, float64)."""
    return sum(((r + 1 + i0) ** (1 - a) - (r + i0) ** (1 - a)) / (hi - lo) for a, lo, hi in laws) / len(laws)


def _sizes(c):
    """Expected n_0..n_L and E_0..E_{L-1} of one batch: the chance of every rank to be in the batch
    after each hop, on a grid of ranks."""
    i0, laws = _laws(c)
    n = c["nodes"]
    edge = np.unique(np.concatenate([np.arange(min(n, 512)), np.geomspace(1, n, 3000).astype(np.int64), [0, n]])).astype(np.float64)
    lo, width = edge[:-1], np.diff(edge)
    p = _prob((lo + edge[1:] - 1) / 2, i0, laws)
    deg = c["edges"] * p
    q = np.full(len(p), min(1.0, c["seeds"] / n))
    ns, es = [float(c["seeds"])], []
    for d in _fans(c):
        take = deg if d < 0 else np.minimum(deg, d)
        e = float(np.sum(width * q * take))
        q = 1 - (1 - q) * np.exp(-e * p)
        es.append(e)
        ns.append(float(np.sum(width * q)))
    return ns, es


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 16 + salt)


def _graph(c, seed):
    n, m = c["nodes"], c["edges"]
    i0, laws = _laws(c)
    gen = _gen(seed, 1)
    perm = torch.randperm(n, device=DEV, generator=gen)  # rank -> node
    step = 1 << 27
    deg = torch.empty(n, dtype=torch.int32, device=DEV)
    for r0 in range(0, n, step):
        r = torch.arange(r0, min(n, r0 + step), device=DEV, dtype=torch.float64)
        want = _prob(r, i0, laws) * m + torch.rand(r.numel(), device=DEV, dtype=torch.float64, generator=gen)
        deg[perm[r0:r0 + r.numel()]] = want.to(torch.int32)
    indptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=indptr[1:])
    del deg
    edges = int(indptr[-1])
    indices = torch.empty(edges, dtype=torch.int32, device=DEV)
    perm = perm.to(torch.int32)
    for e0 in range(0, edges, step):
        k = min(step, edges - e0)
        # an edge takes one of the laws at random
        at = [0, k] if len(laws) == 1 else [0, k // 2, k]
        rank = torch.rand(k, device=DEV, dtype=torch.float64, generator=gen)
        for (a, lo, hi), i, j in zip(laws, at[:-1], at[1:]):
            rank[i:j].mul_(hi - lo).add_(lo).pow_(1.0 / (1.0 - a)).sub_(i0)
        if len(laws) == 2:  # both laws within every row: halves dealt alternately
            h = k // 2
            mixed = torch.empty_like(rank)
            mixed[0:2 * h:2], mixed[1:2 * h:2] = rank[:h], rank[h:2 * h]
            mixed[2 * h:] = rank[2 * h:]
            rank = mixed
        torch.index_select(perm, 0, rank.to(torch.int64).clamp_(0, n - 1), out=indices[e0:e0 + k])
        del rank
    return indptr, indices


def _features(nodes, dim, dtype, seed):
    x = torch.empty((nodes, dim), dtype=DTYPES[dtype], device=DEV)
    gen = _gen(seed, 2)
    return x.random_(0, 256, generator=gen) if dtype == "u8" else x.normal_(generator=gen)


def _seed_lists(c, seed):
    """Distinct nodes; the last of several batches is a partial one."""
    k, b = c["seeds"], c["batches"]
    sizes = [k] * (b - 1) + [k if b == 1 else max(1, k - k // 7)]
    gen = _gen(seed, 3)
    some = torch.randperm(c["nodes"], device=DEV, generator=gen)[:k * b].to(torch.int32)
    return [some[i * k:i * k + s].contiguous() for i, s in enumerate(sizes)]


def _outputs(g, c, fan):
    """Buffers of one launch set as alloc_output makes them, the feature rows and the counts of all its
    batches side by side.  They start as zeros, so that what a batch does not fill is the same everywhere."""
    edge_cap = None
    if min(fan) < 0:  # no hop has more samples than the graph has edges, give or take the rounding of the degrees
        edge_cap = [c["edges"] + c["nodes"]] * len(fan)
    outs = [smfg.alloc_output(g, c["seeds"], fan, edge_capacity=edge_cap, with_features=False) for _ in range(c["batches"])]
    L = len(fan)
    feats = torch.zeros((len(outs), outs[0].node_capacity, c["dim"]), dtype=DTYPES[c["dtype"]], device=DEV)
    counts = torch.zeros((len(outs), 2 * L + 2), dtype=torch.int64, device=DEV)
    for i, o in enumerate(outs):
        for t in o.indptr + o.indices + [o.node_ids]:
            t.zero_()
        if o.labels is not None:
            o.labels.zero_()
        o.features, o.counts = feats[i], counts[i]
        o.c.features, o.c.counts = feats[i].data_ptr(), counts[i].data_ptr()
    return outs, feats, counts


# ---- prepare / run -------------------------------------------------------------------------------

def prepare(case, seed):
    return {"sample": _prepare_sample, "epoch": _prepare_epoch, "gather": _prepare_gather,
            "aggregate": _prepare_block, "layer": _prepare_block}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _keys(case, seed):
    return [(int(seed) << 32) | b for b in range(case["batches"])]


def _prepare_sample(c, seed):
    indptr, indices = _graph(c, seed)
    g = smfg.graph_create(indptr, indices, _features(c["nodes"], c["dim"], c["dtype"], seed))
    if c["labels"]:
        smfg.graph_set_labels(g, torch.randint(0, 172, (c["nodes"],), device=DEV, generator=_gen(seed, 4)))
    fan = _fans(c)
    outs, feats, counts = _outputs(g, c, fan)
    # with whole neighbourhoods a hop's samples are bounded by the graph's edges
    samples = c["edges"] + c["nodes"] if min(fan) < 0 else 0
    wss = [] if c["call"] == "static" else [smfg.workspace_create(g, c["seeds"], fan, 0, samples) for _ in outs]
    result = {"features": feats, "counts": counts}
    for i, o in enumerate(outs):
        result["batch%d" % i] = [o.indptr, o.indices, o.node_ids] + ([o.labels] if o.labels is not None else [])
    return dict(run={"one": _run_one, "many": _run_many, "static": _run_static}[c["call"]], g=g, wss=wss, outs=outs,
                seeds=_seed_lists(c, seed), keys=_keys(c, seed), fan=fan, result=result)


def _run_one(s):
    smfg.sample_mfg(s["g"], s["wss"][0], s["seeds"][0], s["fan"], s["keys"][0], s["outs"][0])
    return s["result"]


def _run_many(s):
    smfg.sample_mfg_many(s["g"], s["wss"], s["seeds"], s["fan"], s["keys"], s["outs"])
    return s["result"]


def _run_static(s):
    smfg.sample_mfg_static(s["g"], s["seeds"][0], s["fan"], s["keys"][0], s["outs"][0])
    return s["result"]


def _weights(dim, out_dim, seed, salt):
    gen = _gen(seed, salt)
    w = (torch.randn((out_dim, 2 * dim), device=DEV, generator=gen) / math.sqrt(2 * dim)).to(torch.float16)
    return w, torch.randn(out_dim, device=DEV, generator=gen) * 0.1


def _widths(c):
    return [c["dim"]] + [c["hidden"]] * (len(_fans(c)) - 1) + [c["classes"]]


def _prepare_epoch(c, seed):
    indptr, indices = _graph(c, seed)
    g = smfg.graph_create(indptr, indices, _features(c["nodes"], c["dim"], c["dtype"], seed))
    fan, widths = _fans(c), _widths(c)
    pipe = BatchPipeline(g, fan, c["seeds"], batches_per_set=c["per_set"])
    rows = smfg.bounds(c["seeds"], fan, c["nodes"])[0]
    model = [_weights(widths[i], widths[i + 1], seed, 8 + i) for i in range(len(fan))]
    hidden = [torch.zeros((rows[len(fan) - 1 - i], widths[i + 1]), dtype=torch.float16, device=DEV) for i in range(len(fan) - 1)]
    logits = [torch.zeros((c["seeds"], c["classes"]), dtype=torch.float32, device=DEV) for _ in range(c["batches"])]
    return dict(run=_run_epoch, pipe=pipe, seeds=_seed_lists(c, seed), keys=_keys(c, seed), rows=rows, hidden=hidden,
                model=[(smfg.sage_pack_weights(w), b) for w, b in model], logits=logits,
                result={"logits": logits, "last_batch": hidden})


def _run_epoch(s):
    done = 0
    for outs in s["pipe"].run(s["seeds"], s["keys"]):
        for o in outs:
            x = o.features
            layers = s["hidden"] + [s["logits"][done]]
            for i, h in enumerate(range(o.L - 1, -1, -1)):
                w, b = s["model"][i]
                smfg.sage_layer(o.indptr[h], o.indices[h], o.counts[h:h + 1], s["rows"][h], x, w, b, h > 0, layers[i])
                x = layers[i]
            done += 1
    return s["result"]


def _prepare_gather(c, seed):
    x = _features(c["nodes"], c["dim"], c["dtype"], seed)
    indptr = torch.zeros(c["nodes"] + 1, dtype=torch.int64, device=DEV)
    g = smfg.graph_create(indptr, torch.zeros(1, dtype=torch.int32, device=DEV)[:0], x)
    ids = torch.randint(0, c["nodes"], (c["rows"],), device=DEV, dtype=torch.int32, generator=_gen(seed, 5))
    out = torch.zeros((c["rows"], c["dim"]), dtype=x.dtype, device=DEV)
    return dict(run=_run_gather, g=g, ids=ids, n=torch.tensor([c["rows"]], device=DEV), rows=c["rows"], out=out)


def _run_gather(s):
    smfg.gather_rows(s["g"], s["ids"], s["n"], s["rows"], s["out"])
    return s["out"]


def _block(c, seed):
    """The outermost block of a batch: rows of up to `fanout` samples, a share `fresh` of them first
    appearances (numbered in order after the destinations), the others known nodes, the popular
    ones more often."""
    gen = _gen(seed, 6)
    dst = c["dst"]
    k = torch.full((dst,), c["fanout"], dtype=torch.int64, device=DEV)
    short = torch.rand(dst, device=DEV, generator=gen) < 0.1
    k[short] = torch.randint(0, c["fanout"], (dst,), device=DEV, generator=gen)[short]
    indptr = torch.zeros(dst + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(k, 0, out=indptr[1:])
    e = int(indptr[-1])
    new = torch.rand(e, device=DEV, generator=gen) < c["fresh"]
    ids = dst - 1 + torch.cumsum(new.to(torch.int64), 0)
    old = (torch.rand(e, device=DEV, dtype=torch.float64, generator=gen).pow_(3) * (ids + 1)).to(torch.int64)
    ids = torch.where(new, ids, torch.minimum(old, ids))
    src = dst + int(new.sum())
    gen = _gen(seed, 7)
    x = torch.empty((src, c["dim"]), dtype=torch.float16 if c["kind"] == "layer" else DTYPES[c["dtype"]], device=DEV)
    return indptr.to(torch.int32), ids.to(torch.int32), x.normal_(generator=gen)


def _prepare_block(c, seed):
    indptr, indices, x = _block(c, seed)
    s = dict(indptr=indptr, indices=indices, x=x, dst=c["dst"], n=torch.tensor([c["dst"]], device=DEV))
    if c["kind"] == "aggregate":
        return dict(s, run=_run_aggregate, out=torch.zeros((c["dst"], c["dim"]), dtype=torch.float32, device=DEV))
    w, b = _weights(c["dim"], c["out_dim"], seed, 8)
    return dict(s, run=_run_layer, w=smfg.sage_pack_weights(w), b=b, relu=c["relu"],
                out=torch.zeros((c["dst"], c["out_dim"]), dtype=DTYPES[c["dtype"]], device=DEV))


def _run_aggregate(s):
    smfg.mean_aggregate(s["indptr"], s["indices"], s["n"], s["dst"], s["x"], s["out"])
    return s["out"]


def _run_layer(s):
    smfg.sage_layer(s["indptr"], s["indices"], s["n"], s["dst"], s["x"], s["w"], s["b"], s["relu"], s["out"])
    return s["out"]


# ---- what the work cannot do without ----------------------------------------------------------------

def _sample_bytes(c):
    n, e = _sizes(c)
    row = c["dim"] * SIZE[c["dtype"]]
    label = 16 * c["seeds"] if c.get("labels") else 0
    # seeds, two row offsets per destination, chosen neighbour ids and feature rows in; blocks, ids and rows out
    return c["batches"] * (4 * n[0] + sum(16 * n[h] + 4 * x for h, x in enumerate(e)) + row * n[-1] + label
                           + sum(4 * n[h] + 4 * x for h, x in enumerate(e)) + (4 + row) * n[-1])


def work(case):
    c = case
    if c["kind"] == "sample":
        return {"bytes": _sample_bytes(c), "flops": 0}
    if c["kind"] == "epoch":
        # preparation, then every layer: block, source rows in, destination rows out
        n, e = _sizes(c)
        widths, moved, flops = _widths(c), _sample_bytes(c), 0.0
        for i, h in enumerate(range(len(e) - 1, -1, -1)):
            moved += c["batches"] * (4 * n[h] + 4 * e[h] + 2 * widths[i] * n[h + 1] + (4 if h == 0 else 2) * widths[i + 1] * n[h])
            flops += c["batches"] * (4.0 * n[h] * widths[i] * widths[i + 1] + e[h] * widths[i])
        return {"bytes": moved, "flops": flops}
    if c["kind"] == "gather":
        return {"bytes": c["rows"] * (4 + 2.0 * c["dim"] * SIZE[c["dtype"]]), "flops": 0}
    edges = c["dst"] * c["fanout"] * 0.95
    rows = c["dst"] + edges * c["fresh"]
    if c["kind"] == "aggregate":
        # the rows that are sampled: nearly all that are not destinations only
        return {"bytes": 4 * c["dst"] + 4 * edges + rows * c["dim"] * SIZE[c["dtype"]] + 4 * c["dst"] * c["dim"], "flops": edges * c["dim"]}
    return {"bytes": 4 * c["dst"] + 4 * edges + rows * c["dim"] * 2 + c["dst"] * c["out_dim"] * SIZE[c["dtype"]] + 4 * c["dim"] * c["out_dim"],
            "flops": 4.0 * c["dst"] * c["dim"] * c["out_dim"] + edges * c["dim"]}


def tolerance(case):
    if case["kind"] in ("sample", "gather"):
        return "exact"
    if case["kind"] == "aggregate":
        return {"rel": 1e-6, "max": 1e-5}  # float sums of up to 64 terms
    # half inputs; the mean is rounded to half once, and so is the result unless it is float
    if case["kind"] == "layer":
        return {"rel": 1e-3, "max": 1e-2}
    return {"rel": 1.2e-3, "max": 1.2e-2}  # two layers of half activations below the logits


# ---- the same in 64 bits -------------------------------------------------------------------------------

def _mean64(indptr, indices, x):
    """Mean of the sampled rows, zeros where nothing was sampled; x in any type, sums in float64."""
    dst = indptr.numel() - 1
    k = (indptr[1:] - indptr[:-1]).to(torch.int64)
    row = torch.repeat_interleave(torch.arange(dst, device=DEV), k)
    out = torch.zeros((dst, x.shape[1]), dtype=torch.float64, device=DEV)
    for c0 in range(0, x.shape[1], 32):
        out[:, c0:c0 + 32].index_add_(0, row, x[:, c0:c0 + 32].to(torch.float64)[indices.to(torch.int64)])
    return out / k.clamp(min=1).to(torch.float64)[:, None]


def _layer64(indptr, indices, x, w, b, relu):
    dst = indptr.numel() - 1
    both = torch.cat([x[:dst].to(torch.float64), _mean64(indptr, indices, x)], 1)
    y = both @ w.to(torch.float64).t() + b.to(torch.float64)
    return y.clamp(min=0) if relu else y


def _mul32(a, m):
    """High and low halves of the 32 x 32 bit product, int64 tensors."""
    p_lo, p_hi = a * (m & 0xFFFF), a * (m >> 16)
    low = p_lo + ((p_hi & 0xFFFF) << 16)
    return (p_hi >> 16) + (low >> 32), low & 0xFFFFFFFF


def _philox(node, hop, slot, key):
    """Word slot % 4 of Philox4x32-10 with counter (node, hop, slot / 4, 0)."""
    c0, c1, c2, c3 = node, torch.full_like(node, hop), torch.full_like(node, slot // 4), torch.zeros_like(node)
    k0, k1 = key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    for _ in range(10):
        (h0, l0), (h1, l1) = _mul32(c0, 0xD2511F53), _mul32(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return (c0, c1, c2, c3)[slot % 4]


def _plain_blocks(indptr, indices, seeds, fan, key):
    """The documented sampling in plain torch: per hop (indptr, indices), and the node ids."""
    nodes, blocks = seeds.to(torch.int64), []
    for h, d in enumerate(fan):
        n = nodes.numel()
        a = indptr[nodes]
        deg = indptr[nodes + 1] - a
        drawn = deg > d
        pos = torch.arange(d, device=DEV).expand(n, d).clone()
        for s in range(d):  # Floyd's algorithm, slot by slot
            j = deg - d + s
            t = _mul32_by(_philox(nodes, h, s, key), (j + 1).clamp(min=0))
            hit = (pos[:, :s] == t[:, None]).any(1)
            pos[:, s] = torch.where(drawn, torch.where(hit, j, t), pos[:, s])
        has = torch.arange(d, device=DEV)[None, :] < torch.minimum(deg, torch.full_like(deg, d))[:, None]
        got = indices[(a[:, None] + pos)[has]].to(torch.int64)
        # local ids by first appearance over (known nodes, samples in scan order)
        both = torch.cat([nodes, got])
        uniq, inv = torch.unique(both, return_inverse=True)
        first = torch.full((uniq.numel(),), both.numel(), dtype=torch.int64, device=DEV)
        first.scatter_reduce_(0, inv, torch.arange(both.numel(), device=DEV), "amin")
        order = torch.argsort(first)
        local = torch.empty_like(order)
        local[order] = torch.arange(order.numel(), device=DEV)
        ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        torch.cumsum(has.sum(1), 0, out=ptr[1:])
        blocks.append((ptr, local[inv[n:]]))
        nodes = uniq[order]
    return blocks, nodes


def _mul32_by(word, m):
    """floor(word * m / 2^32) for 32-bit words and m < 2^31, int64 tensors."""
    lo, hi = word & 0xFFFF, word >> 16
    return (hi * m + ((lo * m) >> 16)) >> 16


def exact(case, seed):
    c = case
    if c["kind"] == "aggregate":
        return _mean64(*_block(c, seed))
    if c["kind"] == "layer":
        w, b = _weights(c["dim"], c["out_dim"], seed, 8)
        return _layer64(*_block(c, seed), w, b, c["relu"])
    if c["kind"] != "epoch":
        return None  # whole numbers, and rows copied bit by bit
    indptr, indices = _graph(c, seed)
    feat = _features(c["nodes"], c["dim"], c["dtype"], seed)
    fan, widths = _fans(c), _widths(c)
    model = [_weights(widths[i], widths[i + 1], seed, 8 + i) for i in range(len(fan))]
    result = []
    for seeds, key in zip(_seed_lists(c, seed), _keys(c, seed)):
        blocks, nodes = _plain_blocks(indptr, indices, seeds, fan, key)
        x = feat[nodes]
        for i, h in enumerate(range(len(fan) - 1, -1, -1)):
            x = _layer64(*blocks[h], x, *model[i], h > 0)
        logits = torch.zeros((c["seeds"], c["classes"]), dtype=torch.float64, device=DEV)
        logits[:x.shape[0]] = x
        result.append(logits)
    return {"logits": result, "last_batch": [None] * (len(fan) - 1)}
