"""The sampler's work as its users call it, in cases that can be timed and compared.

A case names a graph (shaped like one of the synthetic datasets of kgsynth, by
its sizes and laws), a way to use it and the sizes of the call.  The graph of a
dataset is made once per process, on the GPU, from a fixed law: a program loads
one knowledge graph and samples many batches of it, so what a seed changes is
the batch (the sampling key and the query ids; for verification the candidates
too; for graph building the triples themselves).

All outputs are whole numbers, and equal bit for bit for equal inputs.
"""
from __future__ import annotations

import math

import torch

import paper_2110_14890_amd as sm

NINE = "1p 2p 3p 2i 3i ip pi 2u up"
NEGATION = "2in 3in inp pin pni"

# entities, relations, candidate triples drawn, Zipf exponents of heads and
# tails (0: uniform), inverse relations added.  Relations are Zipf(1.0)
# except in "tiny" (uniform).  The power laws are continuous (a bounded
# Pareto law of the rank); repeated triples are dropped.
GRAPHS = {
    "tiny": (1_000, 20, 10_100, 0.0, 0.0, True),
    "fb15k237": (15_000, 237, 360_000, 1.1, 0.0, False),
    "fb400k": (400_000, 900, 4_000_000, 1.2, 1.2, False),
    "wikikg2": (2_500_000, 535, 34_000_000, 1.2, 1.2, False),
    "freebase": (86_000_000, 14_800, 1_200_000_000, 1.3, 1.3, False),
}


def listed():
    return [
        # the smallest call in use: a batch of one-hop queries on a graph that
        # fits in cache, as a serving process or an interactive user makes it
        dict(name="tiny_1p_call", graph="tiny", use="sample", types="1p", batch=64, n_neg=16),
        # one training minibatch of the tiny configuration, deepest shape
        dict(name="tiny_3p_batch", graph="tiny", use="sample_into", types="3p", batch=1024, n_neg=32),
        # one training step of the FB15k-237-shaped configuration: all nine
        # shapes, one after the other on the program's stream
        dict(name="fb15k237_step", graph="fb15k237", use="sample_into", types=NINE, batch=512, n_neg=128),
        # one minibatch of the FB400k-shaped configuration
        dict(name="fb400k_2p_batch", graph="fb400k", use="sample_into", types="2p", batch=4096, n_neg=256),
        # evaluation queries with 1,000 filtered negatives each; a ragged batch
        dict(name="fb400k_3p_eval", graph="fb400k", use="sample_into", types="3p", batch=3001, n_neg=1000),
        # one minibatch of the ogbl-wikikg2-shaped configuration
        dict(name="wikikg2_2i_batch", graph="wikikg2", use="sample_into", types="2i", batch=8192, n_neg=256),
        # a training step of the five shapes with negation, side by side on streams
        dict(name="wikikg2_negation_step", graph="wikikg2", use="streams", types=NEGATION, batch=8192, n_neg=256),
        # a minibatch whose queries share one candidate set
        dict(name="wikikg2_ip_shared", graph="wikikg2", use="shared", types="ip", batch=8192, n_neg=512),
        # evaluation: given candidates of given queries verified on a graph
        dict(name="wikikg2_pi_verify", graph="wikikg2", use="verify", types="pi", batch=4096, n_neg=1000),
        # the minibatch of the paper's sampler-speed experiment: a maximum
        # expansion per relation, most positive attempts rejected
        dict(name="freebase_2p_capped", graph="freebase", use="sample_into", types="2p", batch=1024, n_neg=512,
             max_fanout=10),
        # the benchmark's training step: the Freebase-shaped configuration,
        # three shapes side by side on streams
        dict(name="freebase_step", graph="freebase", use="streams", types="3p ip pi", batch=16384, n_neg=512),
        # a program's start: host triples to device graph, and a first batch
        dict(name="fb400k_start", graph="fb400k", use="build", types="1p", batch=1024, n_neg=64),
    ]


def _between(rng, lo, hi):
    """A whole number of [lo, hi], even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    use = rng.choice(["sample", "sample_into", "sample_into", "sample_into", "streams", "shared", "verify", "build"])
    graph = rng.choice(["tiny", "fb15k237", "fb400k", "wikikg2", "wikikg2", "freebase"])
    if use == "build" and graph == "freebase":
        graph = "fb400k"
    shapes = (NINE + " " + NEGATION).split()
    types = " ".join(rng.sample(shapes, rng.randint(2, 3))) if use == "streams" else rng.choice(shapes)
    case = dict(graph=graph, use=use, types=types, batch=_between(rng, 16, 8192), n_neg=_between(rng, 8, 1000))
    if use == "build":
        case.update(batch=_between(rng, 16, 1024), n_neg=_between(rng, 8, 128))
    elif use != "verify" and rng.random() < 0.15:
        case["max_fanout"] = rng.choice([10, 30, 100, 300])
    while case["batch"] * case["n_neg"] * len(types.split()) > 2 * 16384 * 512:
        case["batch"] //= 2
    return case


# ----------------------------------------------------------------- graphs
def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _rank(u, n, s):
    """Ranks 0 .. n - 1 from uniform u in [0, 1): power law of exponent s."""
    if s == 0.0:
        k = u * n
    elif s == 1.0:
        k = torch.pow(float(n + 1), u) - 1.0
    else:
        k = torch.pow(1.0 - u * (1.0 - float(n + 1) ** (1.0 - s)), 1.0 / (1.0 - s)) - 1.0
    return k.to(torch.int64).clamp_(0, n - 1)


def _candidates(graph, seed, at, count):
    """Candidate triples [at, at + count): entity ids are scattered ranks,
    the same scattering for heads and tails."""
    V, R, _, head_s, tail_s, _ = GRAPHS[graph]
    gen = torch.Generator(device="cuda").manual_seed(1_000_003 * seed + at)
    u = torch.rand((3, count), dtype=torch.float64, device="cuda", generator=gen)
    h = _rank(u[0], V, head_s) * 2654435761 % V
    r = _rank(u[1], R, 0.0 if graph == "tiny" else 1.0)
    t = _rank(u[2], V, tail_s) * 2654435761 % V
    return h, r, t


def _triples(graph, seed):
    """Distinct triples on the GPU, int32 [E, 3]: of the candidates that fall
    into one slot of a hash table the first is kept."""
    n = GRAPHS[graph][2]
    mask = (1 << min(31, (8 * n - 1).bit_length())) - 1
    table = torch.full((mask + 1,), 2**31 - 1, dtype=torch.int32, device="cuda")
    step = 1 << 26
    kept = []
    for keep in (False, True):
        for at in range(0, n, step):
            count = min(step, n - at)
            h, r, t = _candidates(graph, seed, at, count)
            slot = (h * 65537 + r) * _signed(0x9E3779B97F4A7C15) ^ t * _signed(0xC2B2AE3D27D4EB4F)
            slot = (slot ^ (slot >> 32)) * _signed(0xD6E8FEB86659FD93)
            slot = (slot >> 24) & mask
            index = torch.arange(at, at + count, dtype=torch.int32, device="cuda")
            if keep:
                first = table[slot] == index
                kept.append(torch.stack([h[first], r[first], t[first]], dim=1).to(torch.int32))
            else:
                table.scatter_reduce_(0, slot, index, "amin")
    return torch.cat(kept)


_graphs = {}


def _graph(name):
    if name not in _graphs:
        V, R, _, _, _, inverse = GRAPHS[name]
        triples = _triples(name, 0).cpu().numpy()
        torch.cuda.empty_cache()
        _graphs[name] = sm.Graph(triples, V, R, add_inverse=inverse)
    return _graphs[name]


# ------------------------------------------------------------------ cases
def prepare(case, seed):
    use, batch, n_neg = case["use"], case["batch"], case["n_neg"]
    state = {"use": use, "batch": batch, "n_neg": n_neg, "seed": seed, "types": case["types"].split()}
    state["options"] = {"max_fanout": case.get("max_fanout", 0)}
    state["offset"] = offset = (seed * 2654435761 % 10_007) * batch
    if use == "build":
        V, R, _, _, _, inverse = GRAPHS[case["graph"]]
        state["triples"] = _triples(case["graph"], seed + 1).cpu().numpy()
        state["shape"] = (V, R, inverse)
        return state
    graph = state["graph"] = _graph(case["graph"])
    args = sm.make_args(batch, n_neg, seed=seed, query_offset=offset, **state["options"])
    state["calls"] = []
    for qt in state["types"]:
        dag = sm.query_preset(qt)
        if use == "shared":
            out = sm.alloc_shared_outputs(batch, n_neg)
        else:
            out = sm.alloc_outputs(batch, n_neg)
        stream = torch.cuda.Stream() if use == "streams" else None
        state["calls"].append((dag, args, out, stream, sm.Workspace()))
    if use == "verify":
        # the queries of a test set, each with its positive and random
        # entities as candidates
        dag, args, out, _, _ = state["calls"][0]
        sm.sample_positives(graph, dag, args, out)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        candidates = torch.randint(0, graph.V, (batch, n_neg), dtype=torch.int32, device="cuda", generator=gen)
        candidates[:, 0] = out["positive"]
        state["queries"] = (out["anchors"], out["relations"], candidates)
    return state


def run(state):
    use = state["use"]
    if use == "build":
        V, R, inverse = state["shape"]
        state["graph"] = graph = sm.Graph(state["triples"], V, R, add_inverse=inverse)
        return sm.sample(graph, state["types"][0], state["batch"], state["n_neg"], seed=state["seed"])
    graph = state["graph"]
    if use == "sample":
        return sm.sample(graph, state["types"][0], state["batch"], state["n_neg"], seed=state["seed"],
                         query_offset=state["offset"], **state["options"])
    if use == "verify":
        dag, _, _, _, workspace = state["calls"][0]
        anchors, relations, candidates = state["queries"]
        return sm.verify(graph, dag, anchors, relations, candidates, workspace=workspace)
    if use == "shared":
        dag, args, out, _, workspace = state["calls"][0]
        return sm.sample_shared_into(graph, dag, args, out, workspace=workspace)
    if use == "streams":
        here = torch.cuda.current_stream()
        for dag, args, out, stream, workspace in state["calls"]:
            stream.wait_stream(here)
            sm.sample_into(graph, dag, args, out, stream=stream, workspace=workspace)
        for _, _, _, stream, _ in state["calls"]:
            here.wait_stream(stream)
        return [out for _, _, out, _, _ in state["calls"]]
    for dag, args, out, _, workspace in state["calls"]:
        sm.sample_into(graph, dag, args, out, workspace=workspace)
    return [out for _, _, out, _, _ in state["calls"]]


_HOPS = {"1p": 1, "2p": 2, "3p": 3, "2i": 2, "3i": 3, "ip": 3, "pi": 3, "2u": 2, "up": 3,
         "2in": 2, "3in": 3, "inp": 3, "pin": 3, "pni": 3}
_LINE = 64
_EDGES = {"tiny": 19_000, "fb15k237": 310_000, "fb400k": 2_500_000, "wikikg2": 17_600_000, "freebase": 336_000_000}


def _graph_bytes(name):
    """Adjacency of both directions: node pointers, neighbours, and about a
    (relation, first edge) pair per two edges."""
    return 2 * (4 * GRAPHS[name][0] + 4 * _EDGES[name] + 4 * _EDGES[name])


def work(case):
    """Bytes only (the path is whole-number gathers): every output written
    once, given candidates and triples read once, and of the graph one line
    for each candidate tested and three for each hop of a query's grounding
    (node pointer, group, neighbour), but no more than the graph holds."""
    batch, n_neg = case["batch"], case["n_neg"]
    moved = 0
    for qt in case["types"].split():
        tested = batch * n_neg
        if case["use"] == "shared":
            moved += batch * (9 * 4 + n_neg / 8)
        elif case["use"] == "verify":
            moved += batch * (7 * 4 + n_neg / 8 + 4 * n_neg)
        else:
            moved += batch * (10 * 4 + 4 * n_neg)
        moved += min(_graph_bytes(case["graph"]), _LINE * (tested + 3 * _HOPS[qt] * batch))
    if case["use"] == "build":
        moved += 12 * _EDGES[case["graph"]] + _graph_bytes(case["graph"])
    return {"bytes": moved, "flops": 0}


def tolerance(case):
    return "exact"
