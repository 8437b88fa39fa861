"""The calls whose speed is watched: PagIndex.build, insert, search, search_static and PagSearcher.search over
the sizes that the configurations, the tests and the benchmark of this repository use.

A search case is one call on an index that the program built once and keeps: the index depends on the case alone,
the queries on the seed.  A build or online case makes its index inside the pass, from vectors drawn with the seed.
"""
import math

import torch

from paper_2603_06660_amd import FLAG_FP16_VECTORS, FLAG_PERMUTATION_TRANSFORM, PagIndex

DEV = "cuda:0"

# Index families: how the data is drawn and how it is indexed (the benchmark's configurations; n is the case's own).
#   gmm16: 16 isotropic Gaussians; aniso: variances i^-0.8, unit norm; clustered: the same law around 256 centres;
#   gmm1024: 1024 Gaussians and queries of which a tenth lie nowhere near the data; mixture: 64 Gaussians that overlap
#   (well separated ones leave a short search now and then in the wrong one, and the distances say nothing then)


def _search(name, law, n, d, P, deg, metric, efc, nq, K, efs, via="search", half=False, permutation=False):
    case = dict(kind="search", law=law, n=n, d=d, P=P, deg=deg, metric=metric, efc=efc, nq=nq, K=K, efs=efs, via=via,
                half=half, permutation=permutation)
    if name:
        case["name"] = name
    return case


def _grow(name, law, n, d, P, deg, metric, efc, nq, K, efs, rounds, m):
    case = dict(kind="grow", law=law, n=n, d=d, P=P, deg=deg, metric=metric, efc=efc, nq=nq, K=K, efs=efs, rounds=rounds, m=m)
    if name:
        case["name"] = name
    return case


def listed():
    million = ("aniso", 1_000_000, 768, 32, 32, "ip", 500)
    return [
        # one user's question to a serving process: nothing but latency
        _search("one query", *million, nq=1, K=10, efs=64),
        # a handful of questions collected for a few milliseconds, at a length that reaches a high recall
        _search("few queries", *million, nq=37, K=10, efs=512),
        # the batches of 1,000 in which the online experiments of the method's authors come
        _search("thousand queries", *million, nq=1000, K=10, efs=256),
        # the benchmark's step: the whole query set at the operating point of recall 0.95
        _search("whole query set", *million, nq=10_000, K=10, efs=1408),
        # candidate generation for a re-ranker: large K, working set in registers beyond 128 nodes
        _search("thousand neighbours", *million, nq=300, K=1000, efs=4000),
        # the smallest configuration: short rows, L2, searches that stay in the on-chip seen set
        _search("short rows", "gmm16", 10_000, 128, 16, 32, "l2", 100, nq=1000, K=10, efs=64),
        # K = 100 over clustered embeddings, short search, every query of the set
        _search("clustered k100", "clustered", 200_000, 1024, 32, 48, "ip", 200, nq=10_000, K=100, efs=128),
        # cosine with raw inputs, long rows, 64 subspaces, part of the queries out of distribution, an odd batch
        _search("cosine out of distribution", "gmm1024", 200_000, 1536, 64, 48, "cos", 200, nq=777, K=50, efs=768),
        # the 16-bit payload of the method's authors, through the entry point that allocates nothing
        _search("half rows static", "aniso", 200_000, 768, 32, 32, "ip", 200, nq=512, K=10, efs=512, via="static", half=True),
        # the longest rows, through a searcher with its own stream
        _search("longest rows", "aniso", 60_000, 3072, 64, 32, "ip", 200, nq=250, K=10, efs=256, via="searcher", permutation=True),
        # a new index over a mid-sized collection, and its first query batch
        _grow("new index", "aniso", 50_000, 768, 32, 32, "ip", 200, nq=1000, K=10, efs=128, rounds=0, m=0),
        # the online setting: a small index that takes blocks of 1,000 vectors, a query batch after each
        _grow("online blocks", "aniso", 20_000, 384, 16, 32, "l2", 100, nq=1000, K=10, efs=100, rounds=5, m=1000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    law, metric = rng.choice([("aniso", "ip"), ("mixture", "l2"), ("clustered", "ip"), ("mixture", "cos"), ("aniso", "l2")])
    P = rng.choice([8, 16, 24, 32, 48, 64])
    per = rng.choice([4, 8, 12, 16, 20, 24, 32])
    d = min(P * per, 1536 // P * P)
    d = d if d % 4 == 0 else P * 16
    deg = rng.choice([16, 24, 32, 40, 48, 64])
    K = _log(rng, 1, 300)
    if rng.random() < 0.25:
        rounds = rng.choice([0, 0, 2, 3])
        return _grow(None, law, _log(rng, 3000, 30_000), d, P, deg, metric, _log(rng, 60, 300), _log(rng, 16, 2000),
                     min(K, 100), _log(rng, 16, 256), rounds, _log(rng, 64, 2000) if rounds else 0)
    nq, via = _log(rng, 1, 4096), rng.choice(["search", "search", "search", "static", "searcher"])
    if via == "static" and (K > 128 or nq * (2 * d + 16 * 64) > 4_000_000):
        via = "search"
    return _search(None, law, _log(rng, 5000, 100_000), d, P, deg, metric, _log(rng, 60, 300), nq, K, _log(rng, 16, 1024), via=via,
                   half=d % 8 == 0 and rng.random() < 0.2)


# ---- inputs -------------------------------------------------------------------------------------------------


def _rows(case, rows, seed, queries=False):
    """`rows` vectors of the case's law; the centres of a mixture are the law's own, the draws are the seed's."""
    law, d = case["law"], case["d"]
    fixed = torch.Generator(DEV).manual_seed(260306660 + d)
    gen = torch.Generator(DEV).manual_seed(int(seed))
    x = torch.randn(rows, d, generator=gen, device=DEV)
    scale = torch.arange(1, d + 1, device=DEV, dtype=torch.float32) ** -0.4
    if law in ("gmm16", "gmm1024", "mixture"):
        k, spread = {"gmm16": (16, 2.0), "gmm1024": (1024, 2.0), "mixture": (64, 0.5)}[law]
        centres = spread * torch.randn(k, d, generator=fixed, device=DEV)
        away = rows // 10 if queries and law == "gmm1024" else 0
        which = torch.randint(0, k, (rows,), generator=gen, device=DEV)
        x[away:] += centres[which[away:]]
    elif law == "clustered":
        centres = torch.randn(256, d, generator=fixed, device=DEV) * scale
        which = torch.randint(0, 256, (rows,), generator=gen, device=DEV)
        x = centres[which] + 0.5 * x * scale
    else:
        x *= scale
    if case.get("permutation"):
        # an index whose transform is a permutation wants data without preferred axes: spread the variances
        x = x[:, torch.randperm(d, generator=fixed, device=DEV)].contiguous()
    if case["metric"] == "ip" or (law == "aniso" and case["metric"] == "l2"):
        x /= x.norm(dim=1, keepdim=True)
    return x


def _options(case):
    return dict(metric=case["metric"], max_degree=case["deg"], num_subspaces=case["P"], ef_construction=case["efc"], seed=2603)


_indexes, _searchers = {}, {}       # what a serving process keeps: one index per collection, one searcher on it
_INDEX_KEYS = ("law", "n", "d", "P", "deg", "metric", "efc", "half", "permutation")


def _index(case):
    key = tuple(case[k] for k in _INDEX_KEYS)
    if key not in _indexes:
        flags = (FLAG_FP16_VECTORS if case["half"] else 0) | (FLAG_PERMUTATION_TRANSFORM if case["permutation"] else 0)
        _indexes[key] = PagIndex.build(_rows(case, case["n"], 1), flags=flags, **_options(case))
    return key, _indexes[key]


def prepare(case, seed):
    seed = 1_000_003 + int(seed)
    if case["kind"] == "grow":
        return dict(case=case, base=_rows(case, case["n"], 3 * seed), queries=_rows(case, case["nq"], 3 * seed + 1, True),
                    blocks=list(_rows(case, case["rounds"] * case["m"], 3 * seed + 2).split(case["m"])) if case["rounds"] else [])
    key, index = _index(case)
    state = dict(case=case, index=index, queries=_rows(case, case["nq"], seed, True))
    if case["via"] == "searcher":
        if key not in _searchers:
            _searchers[key] = index.searcher()
        state["searcher"] = _searchers[key]
    if case["via"] == "static":     # a caller that cannot allocate owns its result buffers
        state["out"] = (torch.empty(case["nq"], case["K"], dtype=torch.int64, device=DEV),
                        torch.empty(case["nq"], case["K"], dtype=torch.float32, device=DEV))
    return state


def run(state):
    case = state["case"]
    K, efs = case["K"], case["efs"]
    if case["kind"] == "grow":
        index = PagIndex.build(state["base"], capacity=case["n"] + case["rounds"] * case["m"], **_options(case))
        out = [index.search(state["queries"], K, efs)]
        for block in state["blocks"]:
            index.insert(block)
            out.append(index.search(state["queries"], K, efs))
        index.close()
        return out
    if case["via"] == "searcher":
        return [state["searcher"].search(state["queries"], K, efs)]
    if case["via"] == "static":
        return [state["index"].search_static(state["queries"], K, efs, state["out"])]
    return [state["index"].search(state["queries"], K, efs)]


# ---- what a pass cannot do without ---------------------------------------------------------------------------


def _search_work(case, nq, ef, b, deg_fraction=1.0):
    """One adjacency record per expanded node and one stored vector per exact distance, the method's own terms: a
    search expands about max(efS, b) nodes and computes six to eight distances for each (the library's counters on
    the benchmark's configurations: 5.9 to 7.1), plus the b entry nodes."""
    d, P, deg = case["d"], case["P"], case["deg"]
    words = 2 if P <= 16 else 4 if P <= 32 else 8
    record = (((deg * 12 + 15) // 16 * 16 + deg * words * 4) + 127) // 128 * 128
    hops = max(ef, b)
    exact = min(b + 6.5 * hops, case["n"])
    row = d * (2 if case.get("half") else 4)
    return (nq * (4.0 * d + hops * record + exact * row),
            nq * (2.0 * d * d + 32.0 * d + hops * deg * P + exact * 3.0 * d))


def work(case):
    nq, K = case["nq"], case["K"]
    bytes_, flops = _search_work(case, nq, case["efs"], max(10, K))
    bytes_ += nq * 12.0 * K
    if case["kind"] == "grow":
        total = case["n"] + case["rounds"] * case["m"]
        bytes_, flops = bytes_ * (case["rounds"] + 1), flops * (case["rounds"] + 1)
        b2, f2 = _search_work(case, total, case["efc"], min(case["efc"], 100))
        # pruning reads every candidate once, the reverse edges the neighbours of each target once
        rows = total * (case["efc"] + case["deg"]) * 4.0 * case["d"]
        bytes_, flops = bytes_ + b2 + rows, flops + f2 + rows * 0.75 * (1 + case["deg"] / 2)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """Distances are sums in 64 bits rounded once to 32: two correct implementations agree to the last bit in all but a
    few values, and choose the same nodes wherever two distances differ at all.  Against the plain C oracle, which adds
    in another order, all id slots of the benchmark's 10,000 queries agree; the tests allow one id in a thousand."""
    return {"rel": 1e-6, "max": 1e-3, "differ": 1e-3}


# ---- the answer in 64 bits -------------------------------------------------------------------------------------


def _nearest(base, queries, K, metric):
    b, q = base.double(), queries.double()
    if metric == "cos":
        b, q = b / b.norm(dim=1, keepdim=True), q / q.norm(dim=1, keepdim=True)
    bn = (b * b).sum(1)
    out = []
    step = max(1, min(q.shape[0], 2_000_000_000 // (8 * b.shape[0])))
    for s in range(0, q.shape[0], step):
        qq = q[s:s + step]
        dd = torch.addmm(bn[None, :], qq, b.t(), alpha=-2.0) + (qq * qq).sum(1, keepdim=True)
        out.append(torch.topk(dd, K, dim=1, largest=False, sorted=True).values.clamp_min(0.0))
    return torch.cat(out) * (1.0 if metric == "l2" else 0.5)


def exact(case, seed):
    """The distances of the true K nearest neighbours, which the search approximates; which ids these are is left open
    (None): an approximate search may miss some."""
    seed = 1_000_003 + int(seed)
    K, metric = case["K"], case["metric"]
    if case["kind"] == "grow":
        state = prepare(case, seed - 1_000_003)
        base, out = state["base"], []
        for block in [None] + state["blocks"]:
            base = base if block is None else torch.cat([base, block])
            out.append((None, _nearest(base, state["queries"], K, metric)))
        return out
    return [(None, _nearest(_rows(case, case["n"], 1), _rows(case, case["nq"], seed, True), K, metric))]
