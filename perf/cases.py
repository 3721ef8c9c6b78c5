"""Cases that the speed of the framework is measured on.

A case is one call (or one short sequence of calls) that a program makes in
earnest, on a synthetic hypergraph of a stated family.  Kinds:

  query     a stratified graph is at hand; select seeds on it
  pipeline  a hypergraph is at hand in device memory; build the graph,
            stratify it, select seeds (what bench.py calls a step)
  batch     several stratified graphs are at hand; one batched seed selection
  serve     several stratified graphs are at hand; a serving session answers
            a handful of queries on them
  generate  a stratified graph and a device buffer are at hand; fill the
            buffer with a range of RR sets
  greedy    a pool of RR sets is at hand; greedy max coverage over it and the
            coverage of its seeds

Hypergraph families (sizes of hyperedges / popularity of members) are those
of the repository's workloads: "tiny" uniform [2,6] / uniform, "mid"
power law 2.5 on [2,50] / Zipf 1.0, "large" power law 2.2 on [2,200] /
Zipf 1.1, "multi" power law 2.5 on [2,100] / uniform, "serving" power law 2.1
on [2,1000] / uniform; always two hyperedges per vertex, give or take.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2406_01911_amd as hy
from paper_2406_01911_amd import autotune

# hyperedge sizes (law, exponent, smallest, largest) and Zipf exponent of the
# members' popularity (0: uniform)
FAMILIES = {
    "tiny": (("uniform", 0.0, 2, 6), 0.0),
    "mid": (("powerlaw", 2.5, 2, 50), 1.0),
    "large": (("powerlaw", 2.2, 2, 200), 1.1),
    "multi": (("powerlaw", 2.5, 2, 100), 0.0),
    "serving": (("powerlaw", 2.1, 2, 1000), 0.0),
}
MODELS = {"const": hy.MODEL_CONST, "wc": hy.MODEL_WC, "lt_const": hy.MODEL_LT_CONST, "lt_wc": hy.MODEL_LT_WC,
          "layered": hy.MODEL_LAYERED, "gaps_const": hy.MODEL_GAPS_CONST, "gaps_wc": hy.MODEL_GAPS_WC}


def listed():
    base = {"p": 0.0, "eps": 0.1, "tuning": "default"}
    return [
        # the smallest call: an interactive query on a graph of a thousand
        # vertices that is already at hand; launches and waits are what counts
        dict(base, name="tiny_query", kind="query", family="tiny", n=1000, m=2000, model="const", p=0.05, k=10,
             eps=0.5),
        # an odd-sized range of RR sets on an odd-sized graph, starting inside
        # a ladder block: a program that samples by itself
        dict(base, name="small_generate_odd", kind="generate", family="mid", n=10007, m=20011, model="wc", k=1,
             id_begin=513, ids=777, tag=1),
        # the ordinary query, from the hypergraph to the seeds, under the
        # tuning stored for it
        dict(base, name="mid_wc_pipeline", kind="pipeline", family="mid", n=100000, m=200000, model="wc", k=50,
             tuning="mid"),
        # the same hypergraph under linear threshold
        dict(base, name="mid_lt_pipeline", kind="pipeline", family="mid", n=100000, m=200000, model="lt_wc", k=50),
        # a block of RR sets on the ordinary graph, default execution parameters
        dict(base, name="mid_generate", kind="generate", family="mid", n=100000, m=200000, model="wc", k=1,
             id_begin=0, ids=4096, tag=0),
        # a million vertices under linear threshold: mostly graph preparation
        # and greedy
        dict(base, name="large_lt_pipeline", kind="pipeline", family="large", n=1000000, m=2000000, model="lt_wc",
             k=100),
        # ... under the stratified setting
        dict(base, name="large_layered_pipeline", kind="pipeline", family="large", n=1000000, m=2000000,
             model="layered", k=100),
        # ... under the independent cascade, by geometric gaps
        dict(base, name="large_gaps_pipeline", kind="pipeline", family="large", n=1000000, m=2000000,
             model="gaps_const", p=0.01, k=100, tuning="large_gaps"),
        # ... by one coin per channel: bench.py's default workload
        dict(base, name="large_const_pipeline", kind="pipeline", family="large", n=1000000, m=2000000, model="const",
             p=0.01, k=100, tuning="large"),
        # greedy and coverage over sets of tens of thousands of members
        dict(base, name="large_greedy", kind="greedy", family="large", n=1000000, m=2000000, model="const", p=0.01,
             k=100, tuning="large", ids=2048),
        # independent instances of mixed size, p and k in one batch
        dict(base, name="batch_mixed", kind="batch", family="multi", n=10000, n_max=150000, graphs=8, m=2, model="const",
             p=0.005, p_max=0.05, k=10, k_max=200),
        # a serving session: eight queries over four graphs of mixed size
        dict(base, name="serve_mixed", kind="serve", family="serving", n=10000, n_max=100000, graphs=4, m=2, model="wc",
             k=10, k_max=200, queries=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "query", "pipeline", "pipeline", "generate", "greedy", "batch", "serve"])
    c = {"kind": kind, "p": 0.0, "eps": rng.choice([0.1, 0.2, 0.5]), "tuning": "default", "k": _log_int(rng, 5, 200)}
    if kind in ("batch", "serve"):
        c["n"] = _log_int(rng, 5000, 20000)
        c["n_max"] = c["n"] * rng.randint(2, 5)
        c["graphs"] = rng.randint(2, 4)
        c["m"] = 2
        c["k_max"] = min(200, c["k"] * 4)
        if kind == "batch":
            c.update(family="multi", model="const", p=0.005, p_max=round(rng.uniform(0.01, 0.05), 4))
        else:
            c.update(family="serving", model="wc", queries=rng.randint(3, 8))
        return c
    n = _log_int(rng, 1000, 400000)
    c["n"], c["m"] = n, 2 * n + rng.randint(-n // 4, n // 4)
    c["model"] = rng.choice(["const", "wc", "wc", "lt_const", "lt_wc", "layered", "gaps_const", "gaps_wc"])
    c["family"] = rng.choice(["tiny", "mid", "large", "multi"])
    if c["model"].endswith("const"):
        c["p"] = round(rng.uniform(0.005, 0.02), 4)
    if c["model"] == "const" and c["family"] == "large" and n > 100000:
        c["tuning"] = "large"   # supercritical: the setting stored for such graphs
    if kind == "generate":
        c.update(id_begin=_log_int(rng, 1, 5000) - 1, ids=_log_int(rng, 1, min(3000, 200000000 // n)),
                 tag=rng.randint(0, 1), k=1)
    if kind == "greedy":
        c.update(ids=_log_int(rng, 64, 3000))
    return c


def _mean_size(law):
    name, gamma, lo, hi = law
    s = np.arange(lo, hi + 1, dtype=np.float64)
    w = s ** (-gamma) if name == "powerlaw" else np.ones_like(s)
    return float((s * w).sum() / w.sum())


def _hypergraph(n, m, family, seed):
    """he_off, he_mem (int32, on the GPU) of a random hypergraph: sizes by
    inverse CDF, members by popularity over a random permutation, drawn again
    where a hyperedge has one twice."""
    (name, gamma, lo, hi), zipf = FAMILIES[family]
    gen = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)
    f64 = dict(device="cuda", dtype=torch.float64)
    s = torch.arange(lo, hi + 1, **f64)
    cdf = torch.cumsum(s ** (-gamma), 0)
    size = lo + torch.searchsorted(cdf / cdf[-1], torch.rand(m, generator=gen, **f64), right=True).clamp_(max=hi - lo)
    size.clamp_(max=n)
    off = torch.zeros(m + 1, device="cuda", dtype=torch.int64)
    torch.cumsum(size, 0, out=off[1:])
    nnz = int(off[-1])
    if zipf:
        pop = torch.cumsum(torch.arange(1, n + 1, **f64) ** (-zipf), 0)
        pop /= pop[-1].clone()
        perm = torch.randperm(n, generator=gen, device="cuda")

    def members(count):
        if not zipf:
            return torch.randint(0, n, (count,), generator=gen, device="cuda")
        r = torch.searchsorted(pop, torch.rand(count, generator=gen, **f64), right=True)
        return perm[r.clamp_(max=n - 1)]

    seg = torch.repeat_interleave(torch.arange(m, device="cuda"), size, output_size=nnz)
    mem = members(nnz)
    while True:
        key, at = torch.sort(seg * n + mem, stable=True)
        again = at[1:][key[1:] == key[:-1]]
        if again.numel() == 0:
            break
        mem[again] = members(again.numel())
    return off.to(torch.int32), mem.to(torch.int32)


def _graph(hg, n, model, p, tuning):
    g = hy.build_graph(n, hg[0], hg[1], MODELS[model], p)
    info = g.stratify()
    if tuning != "default":
        g.set_tuning(**autotune.load(tuning))
    return g, info


def _instances(case, seed):
    """The graphs of a batch or a session, sizes spread over the logarithm of
    their range."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    out, count = [], case["graphs"]
    for i in range(count):
        x = (i + rng.uniform(0.4, 0.6)) / count
        n = int(round(case["n"] * (case["n_max"] / case["n"]) ** x))
        p = float(np.float32(rng.uniform(case["p"], case.get("p_max", case["p"]))))
        hg = _hypergraph(n, case["m"] * n, case["family"], int(rng.integers(1 << 30)))
        g, _ = _graph(hg, n, case["model"], p, case["tuning"])
        out.append(g)
    return out, rng


def _ks(case, count):
    """k of each query, spread over the case's range."""
    lo, hi = case["k"], case["k_max"]
    return [lo + (hi - lo) * (7 * i % count) // max(count - 1, 1) for i in range(count)]


def prepare(case, seed):
    key = int(seed) % (1 << 32)
    st = {"case": case, "key": key}
    kind, n = case["kind"], case["n"]
    if kind in ("batch", "serve"):
        graphs, rng = _instances(case, seed)
        if kind == "batch":
            st["queries"] = [dict(graph=g, k=k, eps=case["eps"], ell=1.0, seed=key, instance=i)
                             for i, (g, k) in enumerate(zip(graphs, _ks(case, len(graphs))))]
        else:
            pick = [(i if i < len(graphs) else int(rng.integers(len(graphs)))) for i in range(case["queries"])]
            st["queries"] = [(graphs[i], k, case["eps"], 1.0, key, i) for i, k in zip(pick, _ks(case, len(pick)))]
        return st
    st["hg"] = _hypergraph(n, case["m"], case["family"], seed)
    if kind == "pipeline":
        st["tuning"] = case["tuning"]
        return st
    st["g"], _ = _graph(st["hg"], n, case["model"], case["p"], case["tuning"])
    if kind == "generate":
        # the buffer a program keeps for these sets: with constant
        # probabilities a set may reach a giant component
        each = n // 2 if case["model"] in ("const", "gaps_const") else n // 64 + 64
        head = -(-8 * (case["ids"] + 1) // 256) * 256 + -(-4 * case["ids"] // 256) * 256
        st["buf"] = torch.zeros(head // 4 + case["ids"] * each, device="cuda", dtype=torch.int32)
        st["pool"] = hy.Pool(st["g"], buf=st["buf"], id_capacity=case["ids"])
    if kind == "greedy":
        st["pool"] = hy.Pool(st["g"])
        hy.generate_rr(st["g"], key, 0, 0, 0, case["ids"], st["pool"])
    return st


def _answer(r):
    return {f: r[f] for f in ("seeds", "gains", "theta", "rounds", "lambda1", "lambda2", "lambda_u", "entries1",
                              "entries2", "sigma_l", "sigma_u", "spread")}


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "query":
        return _answer(hy.select_seeds(st["g"], case["k"], case["eps"], 1.0, seed=st["key"]))
    if kind == "pipeline":
        g, info = _graph(st["hg"], case["n"], case["model"], case["p"], st["tuning"])
        return {"strata": info, "answer": _answer(hy.select_seeds(g, case["k"], case["eps"], 1.0, seed=st["key"]))}
    if kind == "generate":
        st["pool"].reset()
        hy.generate_rr(st["g"], st["key"], 0, case["tag"], case["id_begin"], case["id_begin"] + case["ids"], st["pool"])
        return st["buf"]
    if kind == "greedy":
        seeds, gains = hy.greedy(st["g"], st["pool"], case["ids"], case["k"])
        return {"seeds": seeds, "gains": gains, "covered": hy.coverage(st["g"], st["pool"], case["ids"], seeds)}
    if kind == "batch":
        rs = hy.select_seeds_batch(st["queries"])
    else:
        sess = hy.Session()
        tickets = [sess.submit(*q) for q in st["queries"]]
        rs, left = [None] * len(tickets), len(tickets)
        while left:
            sess.step()
            for i, t in enumerate(tickets):
                if rs[i] is None:
                    rs[i] = sess.poll(t)
                    left -= rs[i] is not None
        sess.close()
    # the queries' fields side by side: seeds and gains one query after another
    rs = [_answer(r) for r in rs]
    return {f: np.concatenate([np.atleast_1d(np.asarray(r[f])) for r in rs]) for f in rs[0]}


def work(case):
    """Each input read once and each output written once.  How many integer
    operations the coins take depends on the draws, so none are claimed here;
    a few bytes per vertex and incidence stand for the traversal."""
    mean = _mean_size(FAMILIES[case["family"]][0])
    if case["kind"] in ("batch", "serve"):
        count = case["graphs"]
        ns = [case["n"] * (case["n_max"] / case["n"]) ** ((i + 0.5) / count) for i in range(count)]
        incid = sum(case["m"] * n * mean for n in ns)
        edges = sum(case["m"] * n for n in ns)
        return {"bytes": 4 * incid + 4 * edges + 12 * case["k_max"] * case.get("queries", count), "flops": 0}
    read = 4 * (case["m"] + 1) + 4 * case["m"] * mean
    if case["kind"] == "greedy":
        return {"bytes": 12 * case["ids"] + 4 * case["n"] + 12 * case["k"], "flops": 0}
    if case["kind"] == "generate":
        return {"bytes": read + 16 * case["ids"], "flops": 0}
    return {"bytes": read + 12 * case["k"], "flops": 0}


def exact(case, seed):
    """Alpha, beta and theta(l*) of the sample-set layers, by sorting all
    co-member pairs.  Everything else is whole numbers fixed by keyed coins,
    or follows from those."""
    if case["kind"] != "pipeline":
        return None
    n, m = case["n"], case["m"]
    off, mem = _hypergraph(n, m, case["family"], seed)
    off, mem = off.long(), mem.long()
    size = off[1:] - off[:-1]
    # all (v, u) pairs of co-members, u != v
    count = torch.repeat_interleave(size, size)             # per incidence: partners, itself among them
    first = torch.repeat_interleave(off[:-1], size)
    row = torch.repeat_interleave(torch.arange(mem.numel(), device="cuda"), count)
    start = torch.cumsum(count, 0) - count
    partner = first[row] + torch.arange(row.numel(), device="cuda") - start[row]
    pair = mem[row] * n + mem[partner]
    pair = pair[row != partner]
    del row, partner, start, first, count
    pair = torch.sort(pair)[0]
    uniq, w = torch.unique_consecutive(pair, return_counts=True)
    del pair
    v = uniq // n
    deg = torch.bincount(v, minlength=n)
    wmax = int(w.max()) + 1 if w.numel() else 1
    layers, members = torch.unique_consecutive(torch.sort(v * wmax + w)[0], return_counts=True)
    lv = layers // wmax
    l = torch.bincount(lv, minlength=n)
    last = torch.ones_like(lv, dtype=torch.bool)
    last[:-1] = lv[1:] != lv[:-1]                           # the largest weight of v: layer 1
    theta_l = (l.double() / torch.log(l.double() + 1.0).clamp(min=1e-300)).where(l > 0, 0.0).sum() / n
    strata = {"B": None, "sum_top": None, "sum_deg": None, "sum_l": None,
              "alpha": float(members[last].sum()) / max(float(deg.sum()), 1.0), "beta": float(l.sum()) / n,
              "theta_l": float(theta_l)}
    return {"strata": strata, "answer": None}
