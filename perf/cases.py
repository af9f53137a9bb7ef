"""The work that a user of this framework has it do, through its Python entry points, as cases that can be timed.

Kinds of pass (the `kind` of a case):

  step       one chronological batch step of a TGN-style memory model (TigContext.step): scoring a stream, evaluation
  train      a run of consecutive training steps (forward, loss, backward, SGD) and the weights read back at its end,
             as a training loop does between two checkpoints
  modules    one batch step of another instance of the general architecture (TigContext.modules_attach)
  partition  the streaming edge partitioner over an event stream (sep.partition), results on the host
  regroup    what shuffle-and-combine does for one GPU before an epoch: sub-graph of a group of parts, its event
             arrays, a context over them (the temporal adjacency is built here) and the epoch's first step

Graphs are drawn on the GPU: Zipf endpoints by rank, exponential spacings (whole seconds at the configurations' events
per second, so that events share timestamps as they do there), N(0, 1) features, one uniform negative per event, and
the state of a stream's middle (memory rows of the nodes seen so far, time of their last event).  The large graphs keep
their configurations' node counts and event density; the streams are shorter, which a step does not see (it
reads the most recent events of a node).
"""
import math

import numpy as np
import torch

from paper_2308_14129_amd import pac, sep, tig

DEVICE = "cuda:0"

# The graph and model shapes of the five configurations.
TINY = dict(nodes=1000, dst_nodes=0, events=10_000, alpha=1.2, alpha_dst=1.2, per_second=0.1, whole_seconds=False,
            feat=16, mem=32, time=16, emb=32, neighbors=10, heads=2)
MEDIUM = dict(nodes=8227, dst_nodes=1000, events=157_474, alpha=1.1, alpha_dst=1.3, per_second=0.06, whole_seconds=True,
              feat=172, mem=172, time=100, emb=100, neighbors=10, heads=2)
DENSE = dict(nodes=10_000, dst_nodes=984, events=672_447, alpha=1.2, alpha_dst=1.2, per_second=0.26, whole_seconds=True,
             feat=172, mem=172, time=100, emb=100, neighbors=20, heads=2)
MILLION = dict(nodes=1_000_000, dst_nodes=0, events=20_000_000, alpha=1.5, alpha_dst=1.5, per_second=7.7, whole_seconds=True,
               feat=16, mem=100, time=100, emb=100, neighbors=10, heads=2)
PARTITION = dict(nodes=2_600_000, dst_nodes=0, events=32_000_000, alpha=1.6, alpha_dst=1.6, per_second=96.0, whole_seconds=True,
                 feat=8, mem=100, time=100, emb=100, neighbors=10, heads=2)


def listed():
    return [
        # a service that embeds and scores interactions as they arrive, a few at a time: launches and round trips
        dict(MILLION, name="serve_16", kind="step", batch=16, negatives=False, precision="bf16", order="update_first"),
        # evaluation over a small graph with the usual batch of 200
        dict(TINY, name="step_tiny_200", kind="step", batch=200, negatives=True, precision="fp32", order="update_first"),
        # the small datasets' row widths (172 features, 172 state columns)
        dict(MEDIUM, name="step_medium_200", kind="step", batch=200, negatives=True, precision="fp32", order="update_first"),
        # every node has its twenty neighbours: the attention gathers bound the step
        dict(DENSE, name="step_dense_2000", kind="step", batch=2000, negatives=True, precision="bf16", order="update_first"),
        # a million nodes; prediction before the update, as in a training loop's validation
        dict(MILLION, name="step_million_1000", kind="step", batch=1000, negatives=True, precision="bf16", order="deferred"),
        # the headline: one GPU's partition of a billion-edge graph
        dict(PARTITION, name="step_partition_4000", kind="step", batch=4000, negatives=True, precision="bf16", order="update_first"),
        # training on a small dataset
        dict(MEDIUM, name="train_medium_200", kind="train", batch=200, steps=20, order="deferred"),
        # training on a GPU's partition
        dict(PARTITION, name="train_partition_4000", kind="train", batch=4000, steps=20, order="deferred"),
        # the light instances (no neighbours): last message, plain RNN, time projection
        dict(MILLION, name="modules_project_1000", kind="modules", batch=1000, order="update_first", aggregator="last",
             updater="rnn", embedding="time_projection", layers=1, node_feat=False),
        # two attention layers over the 2-hop neighbourhood
        dict(PARTITION, name="modules_two_layers_4000", kind="modules", batch=4000, order="update_first", aggregator="last",
             updater="gru", embedding="attention", layers=2, node_feat=False),
        # cutting a stream into partitions, once per dataset
        dict(MILLION, name="partition_4m", kind="partition", events=4_000_000, parts=8, hubs=0.01),
        # rebuilding a GPU's sub-graph before an epoch
        dict(MILLION, name="regroup_16m", kind="regroup", events=16_000_000, parts=8, group=4, hubs=0.01, batch=1000,
             precision="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["train"] * 3 + ["modules"] * 3 + ["partition", "regroup"])
    nodes = _log_int(rng, 1000, 2_600_000)
    c = dict(kind=kind, nodes=nodes, dst_nodes=0, events=min(32_000_000, max(20_000, _log_int(rng, 8 * nodes, 64 * nodes))),
             alpha=round(rng.uniform(1.1, 1.6), 3), alpha_dst=1.2, per_second=round(math.exp(rng.uniform(math.log(0.05), math.log(100))), 4),
             whole_seconds=rng.random() < 0.8)
    if kind == "partition":
        c.update(events=_log_int(rng, 200_000, 4_000_000), parts=rng.randint(2, 16), hubs=round(rng.uniform(0.002, 0.05), 4))
        return c
    if nodes < 50_000 and rng.random() < 0.5:
        c.update(dst_nodes=_log_int(rng, 200, 2000), alpha_dst=round(rng.uniform(1.1, 1.4), 3))
    heads = rng.choice([1, 2, 2, 2, 4])
    mem = _log_int(rng, 32, 172)
    time = _log_int(rng, 16, 100)
    time += -(mem + time) % heads
    c.update(feat=_log_int(rng, 4, 172), mem=mem, time=time, emb=_log_int(rng, 32, 128), neighbors=rng.randint(5, 20 if heads < 4 else 15),
             heads=heads)
    if kind == "regroup":
        parts = rng.randint(4, 16)
        c.update(events=min(c["events"], 16_000_000), parts=parts, group=parts // 2, hubs=round(rng.uniform(0.002, 0.05), 4),
                 batch=_log_int(rng, 100, 4000), precision=rng.choice(["fp32", "bf16"]), dst_nodes=0)
        c["feat"] = min(c["feat"], 64)
    elif kind == "step":
        c.update(batch=_log_int(rng, 8, 5000), negatives=rng.random() < 0.8, precision=rng.choice(["fp32", "bf16"]),
                 order=rng.choice(["update_first", "update_first", "deferred"]))
    elif kind == "train":
        c.update(batch=_log_int(rng, 100, 4000), steps=20, order=rng.choice(["deferred", "deferred", "update_first"]))
        c["events"] = max(c["events"], 2 * c["batch"] * c["steps"])
    else:
        embedding = rng.choice(["attention", "attention", "identity", "time_projection"])
        layers = rng.choice([1, 2]) if embedding == "attention" else 1
        c.update(batch=_log_int(rng, 100, 4000), order=rng.choice(["update_first", "update_first", "deferred"]),
                 aggregator=rng.choice(["last", "mean"]), updater=rng.choice(["gru", "rnn"]), embedding=embedding, layers=layers,
                 node_feat=rng.random() < 0.3)
        if embedding != "attention":
            c["emb"] = c["mem"]
        if layers == 2:
            c["emb"] += -(c["emb"] + c["time"]) % heads
    c["feat"] = min(c["feat"], max(4, 6_000_000_000 // (4 * c["events"])))
    return c


# --------------------------------------------------------------------------- inputs


def _total_nodes(c):
    return c["nodes"] + c["dst_nodes"]


def _zipf(n, alpha, count, gen):
    cdf = torch.arange(1, n + 1, dtype=torch.float64, device=DEVICE).pow_(-alpha).cumsum_(0)
    u = torch.rand(count, dtype=torch.float64, device=DEVICE, generator=gen) * cdf[-1]
    return torch.searchsorted(cdf, u, out_int32=True).clamp_(max=n - 1)


def _graph(c, gen, features=True, ends=None):
    E, n, ends = c["events"], c["nodes"], ends or gen
    src = _zipf(n, c["alpha"], E, ends)
    if c["dst_nodes"]:
        dst = _zipf(c["dst_nodes"], c["alpha_dst"], E, ends) + n
    else:
        dst = _zipf(n, c["alpha"], E, ends)
        for _ in range(8):
            same = (dst == src).nonzero().flatten()
            if not same.numel():
                break
            dst[same] = _zipf(n, c["alpha"], same.numel(), ends)
        dst = torch.where(dst == src, (src + 1) % n, dst)
    gaps = torch.empty(E, dtype=torch.float64, device=DEVICE).exponential_(c["per_second"], generator=gen)
    ts = gaps.cumsum_(0)
    if c["whole_seconds"]:
        ts.floor_()
    feat = torch.randn((E, c["feat"]), device=DEVICE, generator=gen) if features else None
    return src, dst, ts, feat


def _negatives(c, src, gen):
    if c["dst_nodes"]:
        return torch.randint(c["nodes"], _total_nodes(c), src.shape, dtype=torch.int32, device=DEVICE, generator=gen)
    neg = torch.randint(0, c["nodes"], src.shape, dtype=torch.int32, device=DEVICE, generator=gen)
    return torch.where(neg == src, (neg + 1) % c["nodes"], neg).to(torch.int32)


def _warm_state(c, src, dst, ts, first, gen):
    """Memory rows and last-event times of a stream that has been followed up to event `first`."""
    N = _total_nodes(c)
    last = torch.zeros(N, dtype=torch.float64, device=DEVICE)
    seen = torch.zeros(N, dtype=torch.bool, device=DEVICE)
    for ends in (src[:first].long(), dst[:first].long()):
        last.scatter_reduce_(0, ends, ts[:first], "amax")
        seen[ends] = True
    mem = torch.rand((N, c["mem"]), device=DEVICE, generator=gen) - 0.5
    mem *= seen[:, None]
    return mem, last


def _weights(c, seed):
    """fp32 host weights: Xavier-uniform matrices, biases U(-0.1, 0.1), frequencies a ladder 1 .. 1e-9."""
    r = np.random.default_rng(seed)
    M, T, F, E = c["mem"], c["time"], c["feat"], c["emb"]
    updater, embedding = c.get("updater", "gru"), c.get("embedding", "attention")
    g = 3 * M if updater == "gru" else M
    shapes = {"W_i": (g, 2 * M + T + F), "b_i": (g,), "W_h": (g, M), "b_h": (g,)}
    if embedding == "attention":
        shapes.update(_attention_shapes(M, T, F, E))
    shapes.update({"W_d1": (E, 2 * E), "b_d1": (E,), "w_d2": (E,), "b_d2": (1,)})
    w = {k: _draw_weight(r, k, s) for k, s in shapes.items()}
    w["time_w"] = (10.0 ** (np.arange(T) * (-9.0 / max(T - 1, 1)))).astype(np.float32)
    w["time_b"] = r.uniform(-math.pi, math.pi, T).astype(np.float32)
    if embedding == "time_projection":
        w["time_proj_w"] = r.uniform(-1e-6, 1e-6, M).astype(np.float32)
    return w


def _attention_shapes(width, T, F, E):
    da, dkv = width + T, width + F + T
    return {"W_Q": (da, da), "b_Q": (da,), "W_K": (da, dkv), "b_K": (da,), "W_V": (da, dkv), "b_V": (da,), "W_O": (da, da),
            "b_O": (da,), "W_m1": (E, da + width), "b_m1": (E,), "W_m2": (E, E), "b_m2": (E,)}


def _draw_weight(r, name, shape):
    if name == "w_d2":
        lim = math.sqrt(6.0 / (shape[0] + 1))
    else:
        lim = math.sqrt(6.0 / sum(shape)) if name.startswith("W_") else 0.1
    return r.uniform(-lim, lim, shape).astype(np.float32)


def _context(c, src, dst, ts, feat, weights, nodes, precision="fp32", order="update_first"):
    cfg = tig.make_config(c["mem"], c["time"], c["feat"], c["emb"], c["neighbors"], c["heads"], c["batch"], precision, order)
    return tig.TigContext(cfg, nodes, src, dst, ts, feat, weights, device=DEVICE)


def _parts_of_nodes(c, gen):
    """Node masks as the partitioner leaves them: the hubs (lowest ranks) in every part, the others in one."""
    own = torch.randint(0, c["parts"], (c["nodes"],), device=DEVICE, generator=gen)
    masks = torch.bitwise_left_shift(torch.ones_like(own), own)
    masks[:max(1, int(c["hubs"] * c["nodes"]))] = (1 << c["parts"]) - 1
    return masks


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    s = {"case": c}
    if c["kind"] == "partition":
        s["src"], s["dst"], s["ts"], _ = _graph(c, gen, features=False)
        # the decay spans the stream: the first events weigh about 1 / e^2 of the last
        s["cfg"] = sep.make_config(c["parts"], 2.0 / float(s["ts"][-1]), c["hubs"])
        return s
    if c["kind"] == "regroup":
        # one set of interactions and one cut of its nodes per case, in another chronological order for every seed: the
        # sub-graphs of all seeds have one size
        fixed = torch.Generator(device=DEVICE)
        fixed.manual_seed(c["events"])
        src, dst, ts, feat = _graph(c, gen, ends=fixed)
        order = torch.randperm(c["events"], device=DEVICE, generator=gen)
        src, dst = src[order], dst[order]
        s.update(src=src, dst=dst, ts=ts, feat=feat, weights=_weights(c, seed), masks=_parts_of_nodes(c, fixed))
        s["neg"] = torch.randint(0, c["nodes"] // 8, (c["batch"],), dtype=torch.int32, device=DEVICE, generator=gen)
        return s
    src, dst, ts, feat = _graph(c, gen)
    negatives = c.get("negatives", True)
    first = c["events"] // 2
    weights = _weights(c, seed)
    if c["kind"] == "train":
        ts = ts / 86400.0  # days: the gradients of the frequencies stay of the size of the other weights'
    mem, last = _warm_state(c, src, dst, ts, first, gen)
    s["neg"] = _negatives(c, src, gen) if negatives else None
    if c["kind"] == "modules":
        ctx = _context(c, src, dst, ts, feat, None, _total_nodes(c), order=c["order"])
        r = np.random.default_rng(seed + 1)
        layer2 = None
        if c["layers"] == 2:
            layer2 = {k: _draw_weight(r, k, x) for k, x in _attention_shapes(c["emb"], c["time"], c["feat"], c["emb"]).items()}
        nf = torch.rand((_total_nodes(c), c["mem"]), device=DEVICE, generator=gen) - 0.5 if c["node_feat"] else None
        ctx.modules_attach(weights, c["aggregator"], c["updater"], c["embedding"], nf, c["layers"], layer2)
    else:
        ctx = _context(c, src, dst, ts, feat, weights, _total_nodes(c), c.get("precision", "fp32"), c["order"])
        if c["kind"] == "train":
            ctx.train_attach(weights)
    ctx.state_import(mem, last)
    s.update(ctx=ctx, out=ctx.alloc_outputs(c["batch"], with_neg=negatives), first=first)
    return s


# --------------------------------------------------------------------------- passes


def _next_batch(s):
    """First event of the next batch of the stream; a new epoch begins where less than a batch is left."""
    first, B = s["first"], s["case"]["batch"]
    if first + B > s["case"]["events"]:
        s["ctx"].reset()
        first = 0
    s["first"] = first + B
    return first, (s["neg"][first:first + B] if s["neg"] is not None else None)


def _outputs(out):
    got = {"emb": out.emb, "score_pos": out.score_pos}
    if out.score_neg is not None:
        got["score_neg"] = out.score_neg
    return got


def run(state):
    c = state["case"]
    kind, B = c["kind"], c.get("batch")
    if kind in ("step", "modules"):
        first, neg = _next_batch(state)
        state["ctx"].step(first, B, neg, state["out"])
        return _outputs(state["out"])
    if kind == "train":
        ctx = state["ctx"]
        for _ in range(c["steps"]):
            first, neg = _next_batch(state)
            loss = ctx.train_step(first, B, neg, state["out"], 1e-3)
        return dict(_outputs(state["out"]), loss=loss, weights=ctx.train_get("weights"))
    if kind == "partition":
        return sep.partition(state["cfg"], state["src"], state["dst"], state["ts"], c["nodes"])
    eid, local, n = pac.subgraph(state["src"], state["dst"], state["masks"], (1 << c["group"]) - 1)
    src, dst, ts, feat = pac.gather(state["src"], state["dst"], state["ts"], state["feat"], eid, local)
    ctx = _context(c, src, dst, ts, feat, state["weights"], n, c["precision"])
    out = ctx.alloc_outputs(B)
    ctx.step(0, B, state["neg"], out)
    ctx.close()
    return dict(_outputs(out), eid=eid, local=local, src=src, dst=dst, ts=ts, feat=feat)


# --------------------------------------------------------------------------- what a pass cannot do without


def _distinct(n, alpha, draws):
    """Expected number of distinct values among `draws` Zipf draws of n ranks."""
    p = torch.arange(1, n + 1, dtype=torch.float64).pow_(-alpha)
    p /= p.sum()
    return float((-torch.expm1(draws * torch.log1p(-p.clamp(max=1 - 1e-12)))).sum())


def _ends(c, draws):
    """Expected number of distinct nodes among the endpoints of draws / 2 events."""
    if c["dst_nodes"]:
        return _distinct(c["nodes"], c["alpha"], draws / 2) + _distinct(c["dst_nodes"], c["alpha_dst"], draws / 2)
    return _distinct(c["nodes"], c["alpha"], draws)


def work(case):
    """Expected bytes and flops over the graph's distribution.  A step: every distinct node's row once (endpoints, their
    neighbours, negatives), every distinct (node, time) query's neighbour list and edge features, the rows of the nodes
    with a message and the outputs written; flops of the layers over distinct queries and messages, the attention with
    keys and values folded into the query and output products (the cheaper order for K neighbours)."""
    c = dict(case)
    E, N = c["events"], _total_nodes(c)
    if c["kind"] == "partition":
        return {"bytes": E * (16 + 4) + N * (8 + 1 + 8), "flops": 2.0 * E * 2}
    M, T, F, D, K, H, B = c["mem"], c["time"], c["feat"], c["emb"], c["neighbors"], c["heads"], c["batch"]
    if c["kind"] == "regroup":
        kept = E * 0.8  # most events run between hubs, which every part holds
        graph = E * 8 + N * 8 + N * 4 + kept * (4 + 16 + 4 * F) * 2
        return {"bytes": graph + kept * (2 * 16 + 4 * F) + N * 4 * M / 2, "flops": 1.0 * kept}
    neg = B if c.get("negatives", True) else 0
    winners = _ends(c, 2 * B)
    per_s = c["per_second"]
    pairs = min(2 * B, B / per_s * _ends(c, 2 * per_s)) if c["whole_seconds"] and per_s > 1 else 2 * B
    fill = min(1.0, _ends(c, E) / N * min(1.0, 2 * E / N / K))  # how much of a uniform negative's list is filled
    queries = pairs + neg
    embedding, layers = c.get("embedding", "attention"), c.get("layers", 1)
    slots = (pairs + neg * fill) * K if embedding == "attention" else 0
    rows = min(N, winners + neg + (_ends(c, slots) if slots else 0))
    b = rows * 4 * M + winners * 4 * (M + F + 4) + slots * (16 + 4 * F) + (2 * B + neg) * (4 * D + 4) + B * 24
    msg, gates = 2 * M + T + F, 3 if c.get("updater", "gru") == "gru" else 1
    f = winners * 2 * gates * M * (msg + M) + (B + neg) * 2 * (2 * D * D + D)
    layer = 0.0
    if embedding == "attention":
        da, dkv = M + T, M + F + T
        layer = 2.0 * (da * da + 2 * da * dkv + da * da + D * (da + M) + D * D) + K * H * dkv * 4
        f += queries * layer
        if layers == 2:
            hops = min(_ends(c, slots) * max(1.0, B / max(per_s, 1e-9)) if c["whole_seconds"] and per_s > 1 else slots, slots)
            f += hops * layer
            b += hops * (16 + 4 * F) * K
    weights = sum(int(np.prod(x)) for x in _attention_shapes(M, T, F, D).values()) * layers if embedding == "attention" else 0
    weights += gates * M * (msg + M) + 2 * D * D
    b += 4 * weights
    if c["kind"] == "train":
        b, f = (b + 4 * weights) * c["steps"], 3 * f * c["steps"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] == "partition":
        return {"rel": 1e-9, "differ": 1e-3}  # fp64 sums in any order; a tie of two scores may go either way
    if case["kind"] == "train":
        return {"rel": 1e-4, "max": 2e-2}  # twenty updates apart: sums in any order, now and then a ReLU's zero
    if case.get("precision") == "bf16":
        return {"rel": 1e-4, "max": 1e-2}  # operands as pairs of bf16 values, fp32 sums
    return {"rel": 2e-5, "max": 2e-3}  # 32-bit sums of a few hundred terms in five layers, phases of up to 1e6 rad
