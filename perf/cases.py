"""The calls of this framework that its performance is measured by.

A case is one call, or the few calls that belong together, of a program that prepares GNN mini-batches: the whole
path (directly launched, recorded, recorded for several mini-batches at once), its parts on their own (sampling,
de-duplication, feature gather), batch generation for training, and the set-up of the cache after pre-sampling.  The
shapes are those of the workloads in `workload.py` and of the tests, with the graphs cut down to a few million nodes
so that an input is made in a fraction of a second; batch sizes, fan-outs, row sizes and the shares of the tiers are
the originals'.
"""
import math

import numpy as np
import torch

from paper_2310_00837_amd import helios
from paper_2310_00837_amd import workload as W

DEV = torch.device("cuda", 0)
DTYPES = {"f32": torch.float32, "f16": torch.float16}
BATCH_OPS = ("call", "plan", "gang", "blocks")


def listed():
    return [
        # the smallest whole-path call: the tiny workload (10 k nodes, 128 seeds), launched directly, its misses served
        # by helios_gather_miss right after it.  Launches and latency are all there is.
        {"name": "call-tiny", "op": "call", "nodes": 10_000, "edges": 100_000, "seeds": 128, "fan": "5,5", "dim": 64,
         "dtype": "f32", "hbm": 0.10, "host": 0.20, "draw": "split", "serve": True, "members": 1},
        # the medium workload as a recorded batch that serves its own misses: three tiers, half of the rows over the link
        {"name": "plan-medium", "op": "plan", "nodes": 1_000_000, "edges": 15_000_000, "seeds": 1024, "fan": "10,10",
         "dim": 128, "dtype": "f32", "hbm": 0.10, "host": 0.30, "draw": "split", "serve": True, "members": 1},
        # the paper's shape (fan-outs 25 and 10, 512-byte rows, 20 GB + 30 GB of a 57 GB table) as a gang of four, the
        # form in which a loader keeps the GPU busy
        {"name": "gang-paper", "op": "gang", "nodes": 4_000_000, "edges": 57_600_000, "seeds": 1024, "fan": "25,10",
         "dim": 128, "dtype": "f32", "hbm": 0.35, "host": 0.53, "draw": "split", "serve": False, "members": 4},
        # the tier sweep's end: everything in HBM (288 GB hold the paper's tables whole), skewed seeds with repeats
        {"name": "gang-resident", "op": "gang", "nodes": 4_000_000, "edges": 57_600_000, "seeds": 1024, "fan": "25,10",
         "dim": 128, "dtype": "f32", "hbm": 1.0, "host": 0.0, "draw": "zipf", "serve": False, "members": 4},
        # the wide workload: three hops, 2 KB half-precision rows, most of the table in HBM
        {"name": "plan-wide", "op": "plan", "nodes": 2_000_000, "edges": 40_000_000, "seeds": 1024, "fan": "10,10,10",
         "dim": 1024, "dtype": "f16", "hbm": 0.64, "host": 0.24, "draw": "split", "serve": False, "members": 1},
        # a training step's preparation: recorded batch plus the hops in local numbering; a ragged last batch of an
        # epoch, rows of 400 bytes (100 single-precision features)
        {"name": "blocks-ragged", "op": "blocks", "nodes": 500_003, "edges": 7_300_000, "seeds": 777, "fan": "15,10,5",
         "dim": 100, "dtype": "f32", "hbm": 1.0, "host": 0.0, "draw": "split", "serve": False, "members": 1},
        # evaluation: neighbour sampling alone for a long seed list
        {"name": "sample-long", "op": "sample", "nodes": 4_000_000, "edges": 57_600_000, "seeds": 10_000, "fan": "25,10",
         "draw": "split"},
        # de-duplication alone, a two-hop batch's list of ragged length, by the call that allocates nothing
        {"name": "dedup-ragged", "op": "dedup", "nodes": 1_000_000, "ids": 41_237, "noalloc": True},
        # de-duplication alone, the list of the wide workload at its longest
        {"name": "dedup-large", "op": "dedup", "nodes": 8_000_000, "ids": 1_100_000, "noalloc": False},
        # the feature gather alone: the wide workload's unique list, 2 KB rows, all hits in HBM
        {"name": "gather-wide", "op": "gather", "nodes": 2_000_000, "ids": 243_000, "dim": 1024, "dtype": "f16", "hbm": 1.0,
         "host": 0.0},
        # the feature gather alone for small rows (64 bytes), a ragged list
        {"name": "gather-small-rows", "op": "gather", "nodes": 4_000_000, "ids": 100_003, "dim": 32, "dtype": "f16",
         "hbm": 1.0, "host": 0.0},
        # cache set-up after an epoch of pre-sampling: hotness order of all nodes, then the cache map
        {"name": "cache-setup", "op": "setup", "nodes": 8_000_000, "dim": 16, "dtype": "f16", "hbm": 0.20, "host": 0.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case over the ranges that the listed ones stand for."""
    op = rng.choice(["call", "plan", "plan", "gang", "gang", "blocks", "sample", "dedup", "gather", "gather", "setup"])
    nodes = _log_int(rng, 10_000, 4_000_000)
    if op == "setup":
        return {"op": op, "nodes": _log_int(rng, 20_000, 8_000_000), "dim": 16, "dtype": "f16", "hbm": rng.choice([0.05, 0.2, 0.5]),
                "host": 0.0}
    if op == "dedup":
        noalloc = rng.random() < 0.5
        return {"op": op, "nodes": nodes, "ids": _log_int(rng, 500, 262_144 if noalloc else 1_100_000), "noalloc": noalloc}
    dim, dtype = rng.choice([(32, "f16"), (64, "f32"), (100, "f32"), (128, "f32"), (200, "f16"), (256, "f16"), (512, "f16"),
                             (1024, "f16")])
    if dim == 1024:
        nodes = min(nodes, 2_000_000)
    if op == "gather":
        nodes = max(nodes, 20_000)
        return {"op": op, "nodes": nodes, "ids": _log_int(rng, 1_000, min(243_000, nodes // 2)), "dim": dim, "dtype": dtype,
                "hbm": rng.choice([1.0, 1.0, 1.0, 0.9]), "host": 0.05}
    edges = int(nodes * rng.uniform(8, 20))
    if op == "sample":
        return {"op": op, "nodes": nodes, "edges": edges, "seeds": _log_int(rng, 200, min(10_000, nodes // 4)),
                "fan": rng.choice(["25,10", "10,10", "100", "33,5", "15,10,5"]), "draw": rng.choice(["split", "zipf"])}
    fan = rng.choice(["25,10", "10,10", "5,5", "15,10,5", "10,10,10", "40,4"])
    hbm, host = rng.choice([(1.0, 0.0), (1.0, 0.0), (0.5, 0.5), (0.35, 0.53), (0.64, 0.24), (0.9, 0.05)])
    members = rng.choice([2, 3, 4]) if op == "gang" else 1
    if fan.count(",") > 1:
        members = min(members, 3)
    seeds = _log_int(rng, 100, 1024)
    if dim == 1024 and fan.count(",") > 1:
        members = 1 if op == "plan" else min(members, 2)
        seeds = min(seeds, 500) if members > 1 else seeds
    return {"op": op, "nodes": nodes, "edges": edges, "seeds": min(seeds, nodes // 20), "fan": fan, "dim": dim, "dtype": dtype,
            "hbm": hbm, "host": host, "draw": rng.choice(["split", "split", "zipf"]),
            "serve": hbm + host < 1.0 and rng.random() < 0.5, "members": members}


# ------------------------------------------------------------------ inputs


def _fan(case):
    return [int(f) for f in case["fan"].split(",")]


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _pinned(n, dtype=torch.int64):
    return torch.zeros(n, dtype=dtype, pin_memory=True)


def _graph(case, seed):
    """(spec, graph on the GPU): directed power-law graph, hotness order and splits as the workloads have them."""
    sp = W.WorkloadSpec("case", case["nodes"], case["edges"], case.get("dim", 16), DTYPES[case.get("dtype", "f16")], case["seeds"],
                        _fan(case), 0.10, ("frac", case.get("hbm", 1.0)), ("frac", case.get("host", 0.0)), seeds=case["draw"])
    return sp, W.make_graph(sp, seed, DEV)


def _tier_rows(case):
    n = case["nodes"]
    n_hbm = min(n, int(math.floor(case["hbm"] * n + 1e-9)))
    n_host = min(n - n_hbm, int(math.floor(case["host"] * n + 1e-9)))
    return n_hbm, n_host, n - n_hbm - n_host


def _features(case, rows, gen, pinned):
    """Rows of a tier table, uniform on [-1, 1), as the workloads' features are."""
    t = torch.empty((max(rows, 1), case["dim"]), dtype=DTYPES[case["dtype"]], device=DEV).uniform_(-1.0, 1.0, generator=gen)
    if not pinned:
        return t
    host = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    host.copy_(t)
    return host


def _tables(case, seed):
    gen = _generator(seed)
    rows = _tier_rows(case)
    return [_features(case, r, gen, k > 0) for k, r in enumerate(rows)]


def _popular(n, m, gen):
    """m node IDs drawn from a power law over n nodes (exponent 2.1), as a batch's sampled list holds them."""
    i0, q = 10.0, 1.0 - 1.0 / 1.1
    u = torch.rand(m, dtype=torch.float64, device=DEV, generator=gen)
    at = (i0 ** q + u * ((n + i0) ** q - i0 ** q)) ** (1.0 / q) - i0
    node_of = torch.randperm(n, device=DEV, generator=gen).to(torch.int32)
    return node_of[at.to(torch.int64).clamp_(0, n - 1)]


def _buffers(h, case, n_seeds):
    """The caller's output buffers of one mini-batch, worst case, empty."""
    fan = _fan(case)
    hops = helios.alloc_hops(n_seeds, fan, DEV)
    for hb in hops:
        hb.frontier.zero_(), hb.indptr.zero_(), hb.flat.zero_()
    cap = n_seeds + sum(hb.flat.numel() for hb in hops)
    rows = min(cap, case["nodes"])                    # no batch has more unique nodes than the graph
    ints = lambda n: torch.zeros(n, dtype=torch.int32, device=DEV)  # noqa: E731
    return helios.BatchBuffers(hops=hops, sizes=_pinned(2 * len(fan)), unique=ints(rows), inverse=ints(cap), n_unique=_pinned(1),
                               out=torch.zeros((rows, case["dim"]), dtype=DTYPES[case["dtype"]], device=DEV),
                               miss_pos=ints(rows), miss_id=ints(rows), miss_slot=ints(rows), stats=_pinned(4)), cap


def _args(b):
    return (b.hops, b.sizes, b.unique, b.inverse, b.n_unique, b.out, b.miss_pos, b.miss_id, b.miss_slot, b.stats)


def _prepare_batch(case, seed):
    sp, g = _graph(case, seed)
    tabs = _tables(case, seed + 1)
    rows = _tier_rows(case)
    stream = torch.cuda.Stream(device=DEV) if case["op"] != "call" else None     # a direct caller uses its own stream
    torch.cuda.synchronize()
    ctxs, sets, seeds, rngs = [], [], [], []
    for m in range(case["members"]):
        h = helios.Helios(0, stream=stream)
        h.csr_load(g.offsets, g.indices)
        h.cache_build(g.order, rows[0], rows[1], sp.row_bytes, *tabs)
        bufs, cap = _buffers(h, case, case["seeds"])
        h.reserve(cap)
        sd, rs = W.seed_batch(sp, g, m), W.batch_rng_seed(seed, m)
        if case["serve"] and case["op"] != "call":
            h.set_param(helios.PARAM_SERVE_MISSES, 1)
        torch.cuda.synchronize()
        if case["op"] != "call":
            # a loader's first batch runs directly: the recording takes its grid from that batch's hit counts
            other = W.seed_batch(sp, g, m + case["members"])
            torch.cuda.synchronize()                     # the context's stream does not wait for the one that made them
            h.prepare_batch(other, _fan(case), rs + 1, *_args(bufs))
            h.sync()
            for t in (bufs.unique, bufs.inverse, bufs.miss_pos, bufs.miss_id, bufs.miss_slot, bufs.out):
                t.zero_()
            for hb in bufs.hops:
                hb.frontier.zero_(), hb.indptr.zero_(), hb.flat.zero_()
            torch.cuda.synchronize()
        ctxs.append(h), sets.append(bufs), seeds.append(sd), rngs.append(rs)
    s = {"op": case["op"], "fan": _fan(case), "ctxs": ctxs, "sets": sets, "seeds": seeds, "rngs": rngs, "serve": case["serve"],
         "keep": (g, tabs)}
    if case["op"] in ("plan", "blocks"):
        s["plan"] = ctxs[0].plan_create(case["seeds"], s["fan"], *_args(sets[0]))
    if case["op"] == "gang":
        s["gang"] = helios.Gang(ctxs, case["seeds"], s["fan"], sets)
    if case["op"] == "blocks":
        s["rows"] = [torch.zeros_like(hb.frontier) for hb in sets[0].hops]
        s["cols"] = [torch.zeros_like(hb.flat) for hb in sets[0].hops]
    return s


def prepare(case, seed):
    op = case["op"]
    if op in BATCH_OPS:
        s = _prepare_batch(case, seed)
    elif op == "sample":
        sp, g = _graph(case, seed)
        h = helios.Helios(0)
        h.csr_load(g.offsets, g.indices)
        fan = _fan(case)
        hops = helios.alloc_hops(case["seeds"], fan, DEV)
        for hb in hops:
            hb.frontier.zero_(), hb.indptr.zero_(), hb.flat.zero_()
        h.reserve(case["seeds"] + sum(hb.flat.numel() for hb in hops))
        s = {"op": op, "h": h, "fan": fan, "hops": hops, "sizes": _pinned(2 * len(fan)), "seeds": W.seed_batch(sp, g, 0),
             "rng": W.batch_rng_seed(seed, 0), "keep": g}
    elif op == "dedup":
        n, m = case["nodes"], case["ids"]
        h = helios.Helios(0)
        h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV))
        if not case["noalloc"]:
            h.reserve(m)
        s = {"op": op, "h": h, "ids": _popular(n, m, _generator(seed)), "unique": torch.zeros(m, dtype=torch.int32, device=DEV),
             "inverse": torch.zeros(m, dtype=torch.int32, device=DEV), "n_unique": _pinned(1), "noalloc": case["noalloc"]}
    elif op == "gather":
        ids, order, tabs = _gather_inputs(case, seed)
        n, m = case["nodes"], case["ids"]
        h = helios.Helios(0)
        h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV))
        rows = _tier_rows(case)
        h.cache_build(order, rows[0], rows[1], tabs[0].shape[1] * tabs[0].element_size(), *tabs)
        h.reserve(m)
        miss = [torch.zeros(m, dtype=torch.int32, device=DEV) for _ in range(3)]
        s = {"op": op, "h": h, "ids": ids, "out": torch.zeros((m, case["dim"]), dtype=DTYPES[case["dtype"]], device=DEV),
             "miss": miss, "stats": _pinned(4), "keep": tabs}
    else:
        n = case["nodes"]
        gen = _generator(seed)
        # hotness: how many pre-sampled batches held the node; most nodes never or once, hubs in all of 512
        alpha, i0, c = W._power_law_params(n, 4.0 * n, 2.1)
        rate = (c * (torch.randperm(n, device=DEV, generator=gen).to(torch.float64) + i0) ** (-alpha)).to(torch.float32)
        counts = torch.poisson(rate, generator=gen).clamp_(max=512).to(torch.int32)
        h = helios.Helios(0)
        h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV))
        rows = _tier_rows(case)
        table = _features(case, rows[0], gen, False)
        ids = torch.randperm(n, device=DEV, generator=gen)[:min(n, 20_000)].to(torch.int32)
        s = {"op": op, "h": h, "counts": counts, "order": torch.zeros(n, dtype=torch.int32, device=DEV), "n_hbm": rows[0],
             "table": table, "row_bytes": case["dim"] * 2, "ids": ids,
             "out": torch.zeros((ids.numel(), case["dim"]), dtype=DTYPES[case["dtype"]], device=DEV),
             "miss": [torch.zeros(ids.numel(), dtype=torch.int32, device=DEV) for _ in range(3)], "stats": _pinned(4)}
    torch.cuda.synchronize()
    return s


def _gather_inputs(case, seed):
    """(distinct IDs drawn by popularity, hotness order, tier tables)"""
    n, m = case["nodes"], case["ids"]
    gen = _generator(seed)
    order = torch.randperm(n, device=DEV, generator=gen)
    key = -0.909 * torch.log(torch.arange(n, device=DEV, dtype=torch.float64) + 10.0)
    key -= torch.log(-torch.log(torch.rand(n, dtype=torch.float64, device=DEV, generator=gen).clamp_(1e-12, 1 - 1e-12)))
    ranks = torch.topk(key, m).indices
    ids = order[ranks[torch.randperm(m, device=DEV, generator=gen)]].to(torch.int32)
    return ids, order.to(torch.int32), _tables(case, seed + 1)


# ------------------------------------------------------------------ one pass


def _outputs(b):
    return {"hops": [[hb.frontier, hb.indptr, hb.flat] for hb in b.hops], "sizes": b.sizes, "unique": b.unique,
            "inverse": b.inverse, "n_unique": b.n_unique, "out": b.out, "miss": [b.miss_pos, b.miss_id, b.miss_slot],
            "stats": b.stats}


def run(s):
    op = s["op"]
    if op == "call":
        h, b = s["ctxs"][0], s["sets"][0]
        h.prepare_batch(s["seeds"][0], s["fan"], s["rngs"][0], *_args(b))
        if s["serve"]:
            h.gather_miss(b.miss_pos, b.miss_slot, b.miss_pos.numel(), b.stats[3:4], b.out)
        return _outputs(b)
    if op == "plan":
        s["plan"].launch(s["seeds"][0], s["rngs"][0])
        return _outputs(s["sets"][0])
    if op == "blocks":
        s["plan"].launch(s["seeds"][0], s["rngs"][0])
        s["plan"].make_blocks(s["rows"], s["cols"])
        return {"batch": _outputs(s["sets"][0]), "rows": s["rows"], "cols": s["cols"]}
    if op == "gang":
        s["gang"].launch(s["seeds"], s["rngs"])
        return [_outputs(b) for b in s["sets"]]
    if op == "sample":
        s["h"].sample(s["seeds"], s["fan"], s["rng"], s["hops"], s["sizes"])
        return {"hops": [[hb.frontier, hb.indptr, hb.flat] for hb in s["hops"]], "sizes": s["sizes"]}
    if op == "dedup":
        call = s["h"].dedup_noalloc if s["noalloc"] else s["h"].dedup
        call(s["ids"], s["unique"], s["inverse"], s["n_unique"])
        return {"unique": s["unique"], "inverse": s["inverse"], "n_unique": s["n_unique"]}
    if op == "gather":
        s["h"].gather(s["ids"], s["out"], *s["miss"], s["stats"])
        return {"out": s["out"], "miss": s["miss"], "stats": s["stats"]}
    # the cache set-up, and a first gather through the new map
    h = s["h"]
    h.hotness_order(s["counts"], s["order"])
    h.cache_build(s["order"], s["n_hbm"], 0, s["row_bytes"], s["table"], None, None)
    h.gather(s["ids"], s["out"], *s["miss"], s["stats"])
    return {"order": s["order"], "out": s["out"], "miss": s["miss"], "stats": s["stats"]}


# ------------------------------------------------------------------ what a pass cannot do without


def _weights(n, e):
    """The power law's expected degrees at 4096 ranks spread over 0..n-1, and how many nodes each stands for."""
    alpha, i0, c = W._power_law_params(n, float(e), 2.1)
    edge = np.unique(np.round(np.exp(np.linspace(0.0, math.log(n), 4097))).astype(np.int64))
    lo, hi = np.concatenate([[0], edge[:-1]]), edge
    return c * (0.5 * (lo + hi - 1) + i0) ** (-alpha), (hi - lo).astype(np.float64)


def _distinct(n, e, m, share=1.0):
    """Expected distinct nodes among m draws by in-degree, counting only the hottest `share` of the nodes."""
    w, k = _weights(n, e)
    seen = k * -np.expm1(-m * w / np.sum(w * k))
    return float(np.sum(seen[np.cumsum(k) <= share * n + 0.5]))


def _expected(case):
    """(frontier sizes, sample counts) of the hops, in expectation."""
    n, e = case["nodes"], case["edges"]
    w, k = _weights(n, e)
    fronts, flats, nf = [], [], float(case["seeds"])
    for f in _fan(case):
        fronts.append(nf)
        flats.append(nf * float(np.sum(k * np.minimum(w, f)) / n))
        nf = _distinct(n, e, flats[-1])
    return fronts, flats


def work(case):
    op = case["op"]
    if op == "dedup":
        return {"bytes": 4.0 * case["ids"] * 2 + 4.0 * min(case["ids"], case["nodes"]), "flops": 0}
    if op == "setup":
        n = case["nodes"]
        return {"bytes": 4.0 * n * 2 + 4.0 * n * 2, "flops": 0}              # counts -> order -> map
    item = 4 if case.get("dtype", "f16") == "f32" else 2
    if op == "gather":
        return {"bytes": case["ids"] * (8.0 + 2.0 * item * case["dim"]), "flops": 0}
    fronts, flats = _expected(case)
    # row bounds of every frontier node, its samples, its indptr entry; the samples written
    total = sum(fronts) * (16 + 4 + 8) + sum(flats) * 8
    if op == "sample":
        return {"bytes": total, "flops": 0}
    raw = case["seeds"] + sum(flats)
    uniq = min(_distinct(case["nodes"], case["edges"], raw), raw)
    share = 1.0 if case["serve"] else min(1.0, case["hbm"] + case["host"])
    rows = min(uniq, _distinct(case["nodes"], case["edges"], raw, share))
    total += raw * 4 + uniq * 8 + rows * 2.0 * item * case["dim"]
    if op == "blocks":
        total += 4.0 * (sum(fronts) + sum(flats))
    return {"bytes": total * case["members"], "flops": 0}


def tolerance(case):
    """The path indexes and copies: every output is the same whole number or the same bytes."""
    return "exact"


def exact(case, seed):
    """The gather's rows by plain indexing; the other outputs are whole numbers, or rows chosen by them."""
    if case["op"] != "gather":
        return None
    ids, order, tabs = _gather_inputs(case, seed)
    rows = _tier_rows(case)
    rank = torch.empty(case["nodes"], dtype=torch.int64, device=DEV)
    rank[order.to(torch.int64)] = torch.arange(case["nodes"], device=DEV)
    feats = torch.cat([t[:r].to(DEV) for t, r in zip(tabs, rows)])
    r = rank[ids.to(torch.int64)]
    out = feats[r].to(torch.float64)
    out[r >= rows[0] + rows[1]] = 0.0                       # rows of missing IDs are left as the caller had them
    return {"out": out, "miss": [None, None, None], "stats": None}
