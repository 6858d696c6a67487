"""Work that a user of the sampler has it do, as measurable cases.

A case names an entry (one walk job, a prepared batch, an unprepared batch, a round of served
requests, or a whole one-shot program that builds its graph first), a walk logic, a graph
(R-MAT, generated on the device from the seed) and sizes.  Plans are fixed: an autotuned plan
may differ from run to run and would change the sampled stream.  ``tuned`` plans are what the
autotuner settles on for these graphs (member board, h-proportional or label-conditioned
proposals); ``default`` is ``fw_plan_default()``, what a program runs before it tunes.

Every output is whole numbers (vertices and lengths of seeded walks).
"""
import math
import random

import torch

import paper_2512_00705_amd as fw

DEV = "cuda:0"
N2V, PR, MP = "node2vec", "secondpr", "metapath"


def case(name, entry="walk", logic=N2V, scale=20, edges=16, skew=0.57, n=0, L=80, p=0.5, q=2.0, gamma=0.2,
         weights="f32", strategy="auto", plan="tuned", requests=0):
    """weights: f32, q8 (8-bit codes) or none; n: walkers (0: one per vertex; in a batch or a
    served round the largest query's); edges: R-MAT draws per vertex; requests: queries of a
    batch or of a served round."""
    return {"name": name, "entry": entry, "logic": logic, "scale": scale, "edges": edges, "skew": skew, "n": n,
            "L": L, "p": p, "q": q, "gamma": gamma, "weights": weights, "strategy": strategy, "plan": plan,
            "requests": requests}


def listed():
    return [
        # a short walk for a handful of vertices on a small graph: one request of an online
        # program, where launches and latency are all there is
        case("n2v_small_call", scale=12, edges=8, n=61, L=20, p=2.0, q=0.5),
        # the benchmark's job: a walk corpus with one walker per vertex
        case("n2v_job_scale22", scale=22, L=80),
        # the same kind of job before any tuning: the default plan on a preprocessed graph,
        # without edge index or proposal records, from an odd number of starts
        case("n2v_untuned_scale18", scale=18, n=100003, L=33, p=2.0, q=0.5, plan="default"),
        # 8-bit property weights with the paper's uniform proposals and the edge index
        case("n2v_q8_scale20", scale=20, L=40, weights="q8", plan="uniform"),
        # unweighted walks that favour far vertices (q < 1): the split bound on deep trials
        case("n2v_unweighted_scale20", scale=20, L=50, p=4.0, q=0.25, weights="none", plan="uniform"),
        # reservoir sampling only, the ablation's other kernel: every step scans its row
        case("n2v_reservoir_scale19", scale=19, n=30001, L=40, strategy="rvs", plan="default"),
        # second-order PageRank from two million uniform starts
        case("pagerank2_scale21", logic=PR, scale=21, n=2000003, L=80),
        # MetaPath with label-conditioned proposals, a million uniform starts
        case("metapath_scale22", logic=MP, scale=22, n=1 << 20, L=40),
        # a prepared batch of queries with their own p, q, sizes and lengths, on a skewed graph
        case("batch_scale21", entry="batch", scale=21, skew=0.6, n=16384, L=200, requests=512),
        # a few queries handed over in one call that prepares and launches them
        case("batch_now_scale16", entry="batch_now", scale=16, n=512, L=40, requests=24),
        # a burst of requests to the walk server, half Node2Vec, half MetaPath, until the last
        # result is in host memory
        case("serve_scale20", entry="serve", logic="mixed", scale=20, n=16384, L=100, requests=30),
        # a one-shot program: copy and check the graph, preprocess, edge index, proposal
        # records, then one walk job on it
        case("oneshot_scale20", entry="oneshot", scale=20, L=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    entry = rng.choice(["walk", "walk", "walk", "walk", "batch", "batch_now", "serve", "oneshot"])
    logic = "mixed" if entry == "serve" else rng.choice([N2V, N2V, PR, MP]) if entry != "oneshot" else rng.choice([N2V, PR])
    strategy = "rvs" if entry == "walk" and rng.random() < 0.2 else "auto"
    plan = "default" if strategy == "rvs" else rng.choice(["tuned", "tuned", "uniform", "default"])
    weights = "f32" if entry in ("serve", "oneshot") else rng.choice(["f32", "f32", "f32", "q8", "none"])
    if entry == "serve":
        plan = "tuned"
    # steps the case may take in all: scans and untuned plans cost many times a tuned step
    budget = 2e6 if strategy == "rvs" else 1e7 if plan == "default" or (logic == PR and plan != "tuned") else 5e7
    L = _log_int(rng, 1, 160)
    requests = 0
    if entry in ("batch", "batch_now", "serve"):
        requests = _log_int(rng, 2, {"batch": 400, "batch_now": 64, "serve": 30}[entry])
        n = max(1, min(_log_int(rng, 16, 16384), int(6 * budget / (requests * L))))
    else:
        n = max(1, min(_log_int(rng, 1, 1 << 21), int(budget / L)))
    return case("", entry=entry, logic=logic, scale=rng.randint(8, 18 if plan == "default" else 21),
                edges=rng.choice([4, 8, 16, 24]), skew=rng.choice([0.45, 0.57, 0.6]), n=n, L=L,
                p=rng.choice([0.25, 0.5, 1.0, 2.0, 4.0]), q=rng.choice([0.25, 0.5, 1.0, 2.0, 4.0]),
                gamma=rng.choice([0.0, 0.2, 0.5, 0.9]), weights=weights, strategy=strategy, plan=plan,
                requests=requests)


# ------------------------------------------------------------------------------- inputs
def _mix(x):
    """A 62-bit mix of int64 values (torch has no unsigned shift: the sign is masked away)."""
    m = (1 << 62) - 1
    x = (x ^ ((x & m) >> 29)) * 0x3C79AC492BA7B653
    x = (x ^ ((x & m) >> 32)) * 0x1C69B3F74AC4AE35
    return (x ^ ((x & m) >> 27)) & m


def _rmat(scale, edges, a, seed, labels):
    """CSR of an undirected R-MAT graph on the device: loops and duplicates dropped, vertex ids
    shuffled, rows ascending, weights U(1, 10) and labels 0..4 equal in both directions."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    nv, m = 1 << scale, edges << scale
    b = (1.0 - a) * 0.44
    u = torch.zeros(m, dtype=torch.int32, device=DEV)
    v = torch.zeros(m, dtype=torch.int32, device=DEV)
    r = torch.empty(m, dtype=torch.float32, device=DEV)
    for _ in range(scale):
        r.uniform_(generator=g)
        u.mul_(2).add_(r >= a + b)
        v.mul_(2).add_(((r >= a) & (r < a + b)) | (r >= a + 2 * b))
    del r
    perm = torch.randperm(nv, generator=g, device=DEV)
    u, v = perm[u.long()], perm[v.long()]
    keep = u != v
    lo, hi = torch.minimum(u, v)[keep], torch.maximum(u, v)[keep]
    del u, v, keep
    pair = torch.unique(lo * nv + hi)
    lo, hi = pair // nv, pair % nv
    key = torch.sort(torch.cat([pair, hi * nv + lo])).values
    del pair, lo, hi
    src, col = key // nv, key % nv
    row_ptr = torch.zeros(nv + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.bincount(src, minlength=nv).cumsum(0)
    z = _mix(torch.minimum(src, col) * nv + torch.maximum(src, col) + (seed * 0x9E3779B97F4A7C1 & (1 << 61) - 1))
    h = 1.0 + 9.0 * ((z & 0xFFFFFF).float() * 2.0 ** -24)
    label = ((z >> 24) % 5).to(torch.uint8) if labels else None
    return {"nv": nv, "ne": int(col.numel()), "row_ptr": row_ptr, "col": col.int(), "h": h, "label": label}


def _csr(c, seed):
    t = _rmat(c["scale"], c["edges"], c["skew"], seed, c["logic"] in (MP, "mixed"))
    t["h8"], t["h_scale"] = None, 0.0
    if c["weights"] == "q8":
        t["h_scale"] = 10.0 / 255.0
        t["h8"] = torch.round(t["h"] * 25.5).clamp(1, 255).to(torch.uint8)
    if c["weights"] != "f32":
        t["h"] = None
    return t


class _Handle:
    """A library object freed with the state that holds it, before what it uses (``after``)."""

    def __init__(self, value, free, after=None):
        self.value, self._free, self._after = value, free, after

    def __del__(self):
        torch.cuda.synchronize()
        self._free(self.value)


def _create(t):
    return fw.fw_graph_create(t["nv"], t["ne"], t["row_ptr"], t["col"], t["h"], t["label"], on_device=True,
                              h8=t["h8"], h_scale=t["h_scale"])


def _build(c, g):
    """What a program does once per graph for the plans it will run."""
    fw.fw_graph_preprocess(g)
    if c["plan"] == "default":
        return
    fw.fw_graph_build_index(g)
    if c["plan"] == "tuned" and c["logic"] != MP:
        fw.fw_graph_build_alias(g)
    if c["plan"] == "tuned" and c["logic"] in (MP, "mixed"):
        fw.fw_graph_build_label_alias(g)


def _logic(c, p=None, q=None):
    weighted = c["weights"] != "none"
    if c["logic"] == PR:
        return fw.fw_logic_second_pr(c["gamma"], weighted)
    if c["logic"] == MP:
        return fw.fw_logic_metapath([0, 1, 2, 3, 4], weighted)
    return fw.fw_logic_node2vec(p or c["p"], q or c["q"], weighted)


def _plan(c):
    if c["plan"] == "default":
        return fw.fw_plan_default()
    bound = 0 if c["logic"] == MP else 2 if c["plan"] == "tuned" else 1 if c["logic"] == N2V else 0
    proposal = 0 if c["plan"] == "uniform" else 2 if c["logic"] in (MP, "mixed") else 1
    return fw.fw_plan_default(rho=0.4, bound=bound, proposal=proposal)


def _strategy(c):
    return fw.FW_RVS_ONLY if c["strategy"] == "rvs" else fw.FW_AUTO


def _sizes(c):
    """(n, L) of each query of a batch or served round: sizes log-uniform up to the largest."""
    r = random.Random(c["requests"])
    return [(_log_int(r, 1, c["n"]), r.randint(min(5, c["L"]), c["L"])) for _ in range(c["requests"])]


def prepare(c, seed):
    t = _csr(c, seed)
    nv = t["nv"]
    st = {"c": c, "seed": 1000003 * seed + 42}
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 1)
    if c["entry"] == "oneshot":
        st["csr"] = t
    else:
        st["graph"] = _Handle(_create(t), fw.fw_graph_destroy)
        _build(c, st["graph"].value)
    st["plan"], st["strategy"] = _plan(c), _strategy(c)
    if c["entry"] in ("walk", "oneshot"):
        n = c["n"] or nv
        st["n"], st["logic"] = n, _logic(c)
        st["starts"] = (torch.arange(nv, dtype=torch.int32, device=DEV) if c["n"] == 0 else
                        torch.randint(0, nv, (n,), generator=gen, device=DEV, dtype=torch.int32))
        st["paths"] = torch.empty((n, c["L"] + 1), dtype=torch.int32, device=DEV)
        st["lengths"] = torch.empty(n, dtype=torch.int32, device=DEV)
        return st
    sizes = _sizes(c)
    pq = (0.25, 0.5, 1.0, 2.0, 4.0)
    if c["entry"] == "serve":
        # host data: requests come from outside the device
        starts = [torch.randint(0, nv, (n,), generator=gen, device=DEV, dtype=torch.int32).cpu().numpy() for n, _ in sizes]
        logics = [_logic(dict(c, logic=MP)) if i % 2 else _logic(dict(c, logic=N2V), pq[i % 5], pq[i // 5 % 5])
                  for i in range(len(sizes))]
        st["requests"] = [(lg, s, L, st["seed"] + i) for i, (lg, s, (_, L)) in enumerate(zip(logics, starts, sizes))]
        server = fw.fw_server_create(st["graph"].value, st["plan"], st["strategy"], 1 << 30, 64, 256, 4096)
        st["server"] = _Handle(server, fw.fw_server_destroy, st.pop("graph"))
        return st
    queries, so, po = [], 0, 0
    for i, (n, L) in enumerate(sizes):
        queries.append(fw.fw_query(_logic(c, pq[i % 5], pq[i // 5 % 5]), n, L, st["seed"] + i, so, po, so))
        so += n
        po += n * (L + 1)
    st["queries"] = queries
    st["starts"] = torch.randint(0, nv, (so,), generator=gen, device=DEV, dtype=torch.int32)
    st["paths"] = torch.empty(po, dtype=torch.int32, device=DEV)
    st["lengths"] = torch.empty(so, dtype=torch.int32, device=DEV)
    if c["entry"] == "batch":
        st["batch"] = _Handle(fw.fw_batch_create(st["graph"].value, queries, st["plan"], st["strategy"], st["starts"],
                                                 st["paths"], st["lengths"]), fw.fw_batch_destroy, st["graph"])
    return st


def run(st):
    c = st["c"]
    if c["entry"] == "serve":
        s = st["server"].value
        ids = [fw.fw_server_submit(s, *r) for r in st["requests"]]
        left = set(ids)
        while left:
            left.discard(fw.fw_server_next_done(s, 1000))
        return [fw.fw_server_result(s, i, len(r[1]), r[2])[:2] for i, r in zip(ids, st["requests"])]
    if c["entry"] == "batch":
        fw.fw_batch_launch(st["batch"].value)
    elif c["entry"] == "batch_now":
        fw.fw_batch_run_noalloc(st["graph"].value, st["queries"], st["plan"], st["strategy"], st["starts"], st["paths"],
                                st["lengths"])
    else:
        g = _create(st["csr"]) if c["entry"] == "oneshot" else st["graph"].value
        if c["entry"] == "oneshot":
            _build(c, g)
        fw.fw_walk(g, st["logic"], st["plan"], st["strategy"], st["starts"], st["n"], c["L"], st["seed"], st["paths"],
                   st["lengths"])
        if c["entry"] == "oneshot":
            fw.fw_graph_check(g)  # waits for the walks before the graph goes
            fw.fw_graph_destroy(g)
    return st["paths"], st["lengths"]


def work(c):
    """Per step one vertex record (16 bytes), one edge with its weight (8; 5 with codes, 4
    without) and one path slot; per walker its start and length; a one-shot program also reads
    its graph once and writes its index entry (12) and proposal record (64) per edge.  A
    reservoir step reads every edge of its row: the mean row a walk of these graphs meets."""
    nv = 1 << c["scale"]
    ne = 1.7 * c["edges"] * nv
    edge = {"f32": 8, "q8": 5, "none": 4}[c["weights"]] + (1 if c["logic"] in (MP, "mixed") else 0)
    if c["requests"]:  # log-uniform sizes up to n, uniform lengths up to L
        walkers = c["requests"] * max(1.0, c["n"] / max(1.0, math.log(c["n"] + 1)))
        steps = walkers * c["L"] / 2
    else:
        walkers = c["n"] or nv
        steps = walkers * c["L"] * 0.6  # four in ten vertices of such a graph are isolated
    row = 1.0
    if c["strategy"] == "rvs":
        row = min(4000.0, 40.0 * 1.23 ** (c["scale"])) if c["skew"] > 0.5 else 2.0 * c["edges"]
    b = steps * (16 + edge * row + 4) + 8 * walkers
    if c["entry"] == "oneshot":
        b += ne * (8 + 12 + 64) + nv * 24
    return {"bytes": b, "flops": 0}
