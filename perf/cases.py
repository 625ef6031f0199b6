"""The workloads this package is measured on: neighbor sampling, random walks, layer sampling, multi-dimensional
random walks and the request server, each through its public entry point, from a call of one small instance to
thousands of instances.

Every graph is a seeded R-MAT graph (a=.57, b=.19, c=.19) with shuffled vertex ids, sorted lists and edge weights equal to
the out-degree of the destination, built on the GPU and kept resident for the life of the process, as a program keeps the
graph that it samples:

* ``tiny``    scale 12, 65,536 edge draws;
* ``social``  scale 22, edge factor 16 (the sampling workloads);
* ``large``   scale 24, edge factor 16, symmetrised (walks, node2vec and serving; its walk tables are far larger than the caches).

Every output is a vertex id, an offset or a count, so results are whole numbers.
"""
import math
import random

import numpy as np
import torch

from paper_2009_09103_amd import csaw

FANOUT_ROWS = ([10, 5], [25, 10], [15, 10, 5])
_GRAPHS = {"tiny": (12, 1 << 16, False, 12), "social": (22, 16 << 22, False, 22), "large": (24, 16 << 24, True, 24)}
_resident = {}  # graph name -> (csaw.Graph, vertices with an incident edge): at most the three graphs above
_servers = {}   # graph name -> csaw.Server


def listed():
    return [
        # the smallest call: one instance of 256 seeds on a graph that fits the caches; launches and host latency
        {"name": "sample_tiny", "kind": "sample", "graph": "tiny", "instances": 1, "seeds": 256, "spread": 0.0,
         "fanouts": "10,5", "bias": "uniform", "burn": 0.0, "own_out": False},
        # a training minibatch: 1,024 seeds, three unbiased layers, new output arrays for every batch
        {"name": "sample_minibatch", "kind": "sample", "graph": "social", "instances": 1, "seeds": 1024, "spread": 0.0,
         "fanouts": "15,10,5", "bias": "uniform", "burn": 0.0, "own_out": False},
        # one large degree-biased instance, the paper's biased neighbor sampling
        {"name": "sample_degree", "kind": "sample", "graph": "social", "instances": 1, "seeds": 8192, "spread": 0.0,
         "fanouts": "25,10,5", "bias": "neighbor_degree", "burn": 0.0, "own_out": True},
        # a few uneven edge-weighted instances, odd sizes
        {"name": "sample_weighted_few", "kind": "sample", "graph": "social", "instances": 37, "seeds": 301, "spread": 1.0,
         "fanouts": "25,10", "bias": "edge_weight", "burn": 0.0, "own_out": False},
        # thousands of uneven instances in one call, half unbiased and half degree-biased, fanout rows of their own
        {"name": "sample_batched", "kind": "sample", "graph": "social", "instances": 4096, "seeds": 256, "spread": 1.0,
         "fanouts": "rows", "bias": "mixed", "burn": 0.0, "own_out": True},
        # layer sampling: 2,000 instances of 512 seeds, 64 picks a layer
        {"name": "layer_degree", "kind": "layer", "graph": "social", "instances": 2000, "seeds": 512, "fanouts": "64,64",
         "bias": "neighbor_degree"},
        # DeepWalk corpus generation: unbiased walks by the hundred thousand
        {"name": "walk_uniform", "kind": "walk", "graph": "large", "walkers": 1 << 20, "length": 80, "bias": "uniform",
         "restart": 0.0},
        # edge-weighted walks, as many as one served batch
        {"name": "walk_weighted", "kind": "walk", "graph": "large", "walkers": 262144, "length": 80, "bias": "edge_weight",
         "restart": 0.0},
        # the paper's biased walks: few and long, so one chain of steps sets the time
        {"name": "walk_weighted_long", "kind": "walk", "graph": "large", "walkers": 4000, "length": 2000,
         "bias": "edge_weight", "restart": 0.0},
        # node2vec, return 1, common 2, outward 4
        {"name": "walk_node2vec", "kind": "walk", "graph": "large", "walkers": 65536, "length": 80, "bias": "node2vec",
         "restart": 0.0},
        # the paper's multi-dimensional random walk: 2,000 instances, pools of 2,000, 1,703 edges each
        {"name": "mdrw", "kind": "mdrw", "graph": "social", "instances": 2000, "pool": 2000, "budget": 1703},
        # a burst of mixed requests (60% sampling, 40% weighted walks) through the server, results in host memory
        {"name": "served_burst", "kind": "served", "graph": "large", "requests": 24},
    ]


def _log_int(rng, lo, hi):
    """Log-uniform in [lo, hi], odd about every other time."""
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, x | 1 if rng.random() < 0.5 else x))


def draw(rng):
    kind = rng.choice(["sample", "sample", "sample", "walk", "walk", "walk", "layer", "mdrw", "served"])
    if kind == "sample":
        ni = rng.choice([1, 1, _log_int(rng, 2, 2048)])
        burn = rng.choice([0.0, 0.0, 0.0, 0.7])
        return {"kind": "sample", "graph": rng.choice(["tiny", "social", "social"]), "instances": ni,
                "seeds": _log_int(rng, 16, 8192 if ni == 1 else max(16, min(2048, 400000 // ni))),
                "spread": 0.0 if ni == 1 else 1.0,
                "fanouts": "16,16" if burn else rng.choice(["10,5", "25,10", "15,10,5", "25,10,5", "7,3", "64", "rows"]),
                "bias": "uniform" if burn else rng.choice(["uniform", "edge_weight", "neighbor_degree", "mixed"]),
                "burn": burn, "own_out": ni > 64 or rng.random() < 0.5}
    if kind == "walk":
        bias = rng.choice(["uniform", "edge_weight", "edge_weight", "neighbor_degree", "node2vec", "metropolis_hastings"])
        most = 1 << 20 if bias in ("uniform", "metropolis_hastings") else 65536 if bias == "node2vec" else 262144
        return {"kind": "walk", "graph": "large" if bias in ("node2vec", "edge_weight") else rng.choice(["social", "large"]),
                "walkers": _log_int(rng, 64, most), "length": rng.randint(10, 80), "bias": bias,
                "restart": rng.choice([0.0, 0.0, 0.15])}
    if kind == "layer":
        return {"kind": "layer", "graph": "social", "instances": _log_int(rng, 16, 2000), "seeds": _log_int(rng, 16, 1024),
                "fanouts": rng.choice(["64,64", "32,32,32", "10,5", "63"]),
                "bias": rng.choice(["uniform", "edge_weight", "neighbor_degree"])}
    if kind == "mdrw":
        return {"kind": "mdrw", "graph": "social", "instances": _log_int(rng, 16, 2000), "pool": _log_int(rng, 10, 2000),
                "budget": _log_int(rng, 100, 1703)}
    return {"kind": "served", "graph": "large", "requests": rng.randint(5, 23)}


# ---------------------------------------------------------------- inputs
def _rmat(scale, draws, symmetrize, seed):
    """CSR of a seeded R-MAT graph, built on the GPU: no self-loops, no duplicates, sorted lists, shuffled ids."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n = 1 << scale
    u = torch.zeros(draws, dtype=torch.int64, device="cuda")
    v = torch.zeros_like(u)
    for _ in range(scale):
        r = torch.rand(draws, generator=gen, device="cuda")
        u.mul_(2).add_(r >= 0.76)
        v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    order = torch.randperm(n, generator=gen, device="cuda")
    u, v = order[u], order[v]
    keys = u * n + v
    if symmetrize:
        keys = torch.cat([keys, v * n + u])
    del u, v
    keys = keys.sort().values
    keep = torch.ones_like(keys, dtype=torch.bool)
    keep[1:] = keys[1:] != keys[:-1]
    keep &= (keys // n) != (keys % n)
    keys = keys[keep]
    del keep
    deg = torch.bincount(keys // n, minlength=n)
    col = (keys % n).to(torch.int32)
    del keys
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=rowptr[1:])
    weight = deg.to(torch.int32)[col]
    touched = deg > 0
    touched[col.long()] = True
    return rowptr, col, weight, touched.nonzero().flatten().to(torch.int32)


def _graph(name):
    if name not in _resident:
        rowptr, col, weight, touched = _rmat(*_GRAPHS[name])
        host = [x.cpu().numpy() for x in (rowptr, col, weight)]
        del rowptr, col, weight
        torch.cuda.empty_cache()
        _resident[name] = csaw.Graph(host[0], host[1], host[2].view(np.uint32)), touched
    return _resident[name]


def _server(name):
    if name not in _servers:
        _servers[name] = csaw.Server(_graph(name)[0], num_streams=3, max_batch=256, memory_budget_bytes=12 << 30,
                                     max_batch_walkers=1 << 18, result_pool_bytes=2 << 30)
    return _servers[name]


def _pick(pool, count, gen):
    return pool[torch.randint(0, len(pool), (count,), generator=gen, device="cuda")]


def _sizes(case):
    """Seeds per instance: log-normal around the case's median, in [16, 4,096], where the instances are uneven. They belong
    to the case, the seed vertices to the seed."""
    ni, rng = case["instances"], np.random.default_rng(case["seeds"])
    if case["spread"] == 0.0:
        return np.full(ni, case["seeds"], dtype=np.int64)
    x = np.rint(rng.lognormal(np.log(case["seeds"]), case["spread"], size=ni))
    return np.clip(x, 16, 4096).astype(np.int64)


def _offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)


def _fanouts(case):
    if case["fanouts"] != "rows":
        return np.array([int(x) for x in case["fanouts"].split(",")], dtype=np.int32)
    rng = np.random.default_rng(case["instances"])
    rows = np.zeros((case["instances"], max(len(r) for r in FANOUT_ROWS)), dtype=np.int32)
    for i, c in enumerate(rng.integers(0, len(FANOUT_ROWS), size=case["instances"])):
        rows[i, :len(FANOUT_ROWS[c])] = FANOUT_ROWS[c]
    return rows


def _outputs(s):
    """Output arrays at the call's bound, -1 past the last edge: one shape for every batch of these sizes."""
    return (torch.full((s["capacity"],), -1, dtype=torch.int32, device="cuda"),
            torch.full((s["capacity"],), -1, dtype=torch.int32, device="cuda"),
            torch.empty(s["segments"], dtype=torch.int64, device="cuda"))


def prepare(case, seed):
    g, pool = _graph(case["graph"])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s = {"kind": case["kind"], "graph": g, "seed": seed}
    if case["kind"] == "sample":
        s["offsets"] = _offsets(_sizes(case))
        s["seeds"] = _pick(pool, int(s["offsets"][-1]), gen)
        s["fanouts"] = _fanouts(case)
        s["bias"] = np.arange(case["instances"]) % 2 * csaw.NEIGHBOR_DEGREE if case["bias"] == "mixed" else case["bias"]
        s["burn"] = int(case["burn"] * 2 ** 32)
        s["capacity"] = g.sample_bound(s["offsets"], s["fanouts"], s["bias"])
        s["segments"] = s["fanouts"].shape[-1] * case["instances"] + 1
        s["out"] = _outputs(s) if case["own_out"] else None
    elif case["kind"] == "walk":
        s["starts"] = _pick(pool, case["walkers"], gen)
        s["length"], s["bias"] = case["length"], case["bias"]
        s["restart"] = int(case["restart"] * 2 ** 32)
    elif case["kind"] == "layer":
        # sorted and distinct per instance: one vertex out of each of `seeds` equal ranges of the pool
        ni, k = case["instances"], case["seeds"]
        width = len(pool) // k
        at = torch.arange(k, device="cuda") * width + torch.randint(0, width, (ni, k), generator=gen, device="cuda")
        s["seeds"] = pool[at.flatten()]
        s["offsets"] = _offsets(np.full(ni, k))
        s["fanouts"], s["bias"] = _fanouts(case), case["bias"]
    elif case["kind"] == "mdrw":
        s["offsets"] = _offsets(np.full(case["instances"], case["pool"]))
        s["pool"] = _pick(pool, int(s["offsets"][-1]), gen)
        s["budget"] = case["budget"]
    else:
        s["server"] = _server(case["graph"])
        s["requests"], s["replies"] = [], []
        shape = random.Random(case["requests"])  # the burst's sizes belong to the case, its vertices to the seed
        for i in range(case["requests"]):
            if i % 5 < 3:
                # 64 to 1,024 seeds; the arrays that the reply goes into are the request's own
                k, row = int(round(64 * 16 ** shape.random())), FANOUT_ROWS[shape.randrange(2)]
                seeds = _pick(pool, k, gen).cpu().numpy()
                cap = g.sample_bound([0, k], row)
                s["requests"].append(("sample", seeds, row, csaw.UNIFORM if i % 2 == 0 else csaw.NEIGHBOR_DEGREE))
                s["replies"].append((np.full(cap, -1, dtype=np.int32), np.full(cap, -1, dtype=np.int32)))
            else:
                k, length = int(round(1024 * 64 ** shape.random())), shape.randint(10, 80)
                s["requests"].append(("walk", _pick(pool, k, gen).cpu().numpy(), length, csaw.EDGE_WEIGHT))
                s["replies"].append(None)
    return s


def run(s):
    g, seed = s["graph"], s["seed"]
    if s["kind"] == "sample":
        out = s["out"] or _outputs(s)
        g.sample(s["offsets"], s["seeds"], s["fanouts"], s["bias"], rng_seed=seed, out=out, burn=s["burn"])
        return out
    if s["kind"] == "walk":
        return g.walk(s["starts"], s["length"], s["bias"], rng_seed=seed, node2vec=(1, 2, 4), restart=s["restart"])
    if s["kind"] == "layer":
        return g.layer_sample(s["offsets"], s["seeds"], s["fanouts"], s["bias"], rng_seed=seed)
    if s["kind"] == "mdrw":
        return g.mdrw(s["offsets"], s["pool"], s["budget"], rng_seed=seed)
    server, tickets, out = s["server"], [], []
    for i, (what, ids, shape, bias) in enumerate(s["requests"]):
        submit = server.submit_sample if what == "sample" else server.submit_walk
        tickets.append(submit(ids, shape, bias, rng_seed=seed + i, request_id=i))
    for (what, _, _, _), t, reply in zip(s["requests"], tickets, s["replies"]):
        r = server.wait(t)
        if what == "walk":
            out.append(r.paths)
            continue
        reply[0][:r.num_edges] = r.src
        reply[1][:r.num_edges] = r.dst
        out.append((*reply, r.layer_offsets))
    return out


# ----------------------------------------------------------------- work
# Neighbors a frontier vertex yields for a fanout: the mean of min(fanout, degree), over start vertices (uniform over
# vertices with an edge) and over picked ones (their degrees grow with the bias).
_FIRST = {"tiny": 0.45, "social": 0.35, "large": 0.55}
_LATER = {"tiny": 0.9, "social": 0.85, "large": 0.95}
# shorter of the two lists that a node2vec step compares, ids of 4 bytes
_N2V_SHORTER = 1000.0


def _sample_bytes(graph, seeds, row, weighted):
    total, frontier = 0.0, float(seeds)
    n = float(1 << _GRAPHS[graph][0])
    for layer, k in enumerate(row):
        edges = frontier * k * (_FIRST if layer == 0 else _LATER)[graph]
        # per frontier vertex its id, row offsets and total; per edge the id read and the pair written, and for a
        # weighted pick the prefixes that bracket it
        total += frontier * (20.0 if weighted else 12.0) + edges * (28.0 if weighted else 12.0)
        frontier = n * -math.expm1(-0.3 * edges / n)
    return total


def work(case):
    kind = case["kind"]
    if kind == "sample":
        per = case["seeds"] * math.exp(case["spread"] ** 2 / 2)
        rows = FANOUT_ROWS if case["fanouts"] == "rows" else [[int(x) for x in case["fanouts"].split(",")]]
        rows = [[min(k, 2.33) for k in r] for r in rows] if case["burn"] else rows
        weights = {"uniform": [False], "mixed": [False, True]}.get(case["bias"], [True])
        each = [_sample_bytes(case["graph"], per, r, w) for r in rows for w in weights]
        return {"bytes": case["instances"] * sum(each) / len(each), "flops": 0.0}
    if kind == "walk":
        # row offsets, the picked id, the path entry; weighted: the list's total and the prefixes of the pick
        step = 16.0 + {"uniform": 0.0, "metropolis_hastings": 8.0, "node2vec": 4.0 * _N2V_SHORTER}.get(case["bias"], 24.0)
        return {"bytes": case["walkers"] * (case["length"] * step + 8.0), "flops": 0.0}
    if kind == "layer":
        picks = [int(x) for x in case["fanouts"].split(",")]
        frontiers = [case["seeds"]] + picks[:-1]
        w = 24.0 if case["bias"] != "uniform" else 0.0
        return {"bytes": case["instances"] * sum(f * 24.0 + k * (12.0 + w) for f, k in zip(frontiers, picks)), "flops": 0.0}
    if kind == "mdrw":
        return {"bytes": case["instances"] * (case["pool"] * 12.0 + case["budget"] * 20.0), "flops": 0.0}
    # served: the mean request of either kind, its results copied to host memory
    sampling, walks = -(-case["requests"] * 3 // 5), case["requests"] * 2 // 5
    seeds, walkers = (1024 - 64) / math.log(16), (65536 - 1024) / math.log(64)
    one = sum(_sample_bytes("large", seeds, r, w) for r in FANOUT_ROWS[:2] for w in (False, True)) / 4
    return {"bytes": sampling * one + walks * walkers * 45 * 44.0, "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number that has to be the same: there is no value in more bits."""
    return None
