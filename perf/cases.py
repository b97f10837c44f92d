"""Timed cases: the work that programs give this framework, through its public entry points.

Each case is a dict of plain values.  ``prepare`` builds what a program has in
hand before the call (a context, input graphs on the device or, for the request
loop, in host memory), ``run`` is one call and returns its whole result.  Every
result is made of whole numbers defined bit for bit by (input, n, seed, t0, r,
pl); fields that tell how the work was scheduled or how long it took (rounds,
supersteps of ParES, device times) are not part of it and are left out.

Kinds:
  run      Context.run, r global switches of one simple graph
  class    Context.run_class, the same on directed graphs or graphs with loops / multi-edges
  batch    Context.run_batch, many graphs of uneven sizes in one call
  served   Server, a burst of requests from host memory until all results are back
  es       Context.run_es, the switch-by-switch chain
  mixing   Context.mixing, the autocorrelation diagnostic over either chain
  gen      Context.gen_havel_hakimi and gen_relabel on prescribed degrees, or Context.gen_gnp
"""
import math
import random

import numpy as np
import torch

import paper_2111_03005_amd as gesmc

_COUNTS = ("attempts", "legal", "rej_loop", "rej_exists", "rej_pl")
_HUB_DEGREE = 16000  # the largest degree the device's Havel-Hakimi takes
_THIN = (1, 2, 4, 8, 16, 32, 64)


def listed():
    return [
        # the smallest calls, one after another in a sampling loop: latency counts
        {"name": "run_tiny", "kind": "run", "graph": "gnp", "n": 128, "deg": 8.0, "r": 20, "pl": 0},
        # a small graph, G(1024, 10/1023): the benchmark's small workload
        {"name": "run_small", "kind": "run", "graph": "gnp", "n": 1024, "deg": 10.0, "r": 10, "pl": 0},
        # an ordinary graph of some 1e5 edges, odd vertex count, with P_L > 0 (the aperiodic chain)
        {"name": "run_mid_pl", "kind": "run", "graph": "gnp", "n": 20011, "deg": 11.0, "r": 20, "pl": 1 << 28},
        # power-law degrees, n = 2^20: the benchmark's second workload
        {"name": "run_pld_1m", "kind": "run", "graph": "pld", "n": 1 << 20, "gamma": 2.5, "dmin": 5, "dmax": 1024,
         "r": 20, "pl": 0},
        # the largest single graph, G(2^22, 32/(2^22-1)): the benchmark's headline workload
        {"name": "run_gnp_4m", "kind": "run", "graph": "gnp", "n": 1 << 22, "deg": 32.0, "r": 10, "pl": 0},
        # gamma near 2: hubs, long dependency chains inside a superstep
        {"name": "run_hubs", "kind": "run", "graph": "pld", "n": 1 << 19, "gamma": 2.05, "dmin": 1,
         "dmax": _HUB_DEGREE, "r": 10, "pl": 0},
        # a directed graph
        {"name": "class_directed", "kind": "class", "n": 1 << 20, "deg": 4.0, "cls": gesmc.CLASS_DIRECTED, "r": 10},
        # many graphs of very uneven sizes in one call
        {"name": "batch_512", "kind": "batch", "G": 512, "n_lo": 100, "n_hi": 100000, "r": 20},
        # a burst of requests of the serving recipe
        {"name": "served_48", "kind": "served", "pool": 24, "requests": 48, "n_lo": 1000, "n_hi": 1000000},
        # the switch-by-switch chain, half an expected switch per edge
        {"name": "es_pld_1m", "kind": "es", "n": 1 << 20, "gamma": 2.5, "dmin": 5, "dmax": 1024, "share": 0.5},
        # the mixing diagnostic on a point of the power-law grid
        {"name": "mixing_8k", "kind": "mixing", "n": 1 << 13, "gamma": 2.2, "K": 200, "chain": gesmc.CHAIN_GLOBAL},
        # the power-law input: a simple graph of 2^20 prescribed degrees, its vertices relabelled
        {"name": "gen_pld_1m", "kind": "gen", "graph": "pld", "n": 1 << 20, "gamma": 2.5, "dmin": 5, "dmax": 1024},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "hubs", "class", "batch", "served", "es", "mixing", "gen"])
    if kind == "run":
        if rng.random() < 0.6:
            c = {"kind": "run", "graph": "gnp", "n": _log_int(rng, 100, 1 << 21), "deg": round(rng.uniform(4, 32), 2)}
        else:
            n = _log_int(rng, 1000, 1 << 20)
            c = {"kind": "run", "graph": "pld", "n": n, "gamma": round(rng.uniform(2.1, 3.0), 3),
                 "dmin": rng.randint(2, 5), "dmax": max(8, min(1024, math.isqrt(n)))}
        c["r"] = rng.randint(5, 20)
        c["pl"] = rng.choice([0, 0, 0, 1 << 28])
        return c
    if kind == "hubs":
        return {"kind": "run", "graph": "pld", "n": _log_int(rng, 1 << 16, 1 << 20),
                "gamma": round(rng.uniform(2.03, 2.2), 3), "dmin": 1, "dmax": _HUB_DEGREE, "r": rng.randint(5, 10),
                "pl": 0}
    if kind == "class":
        return {"kind": "class", "n": _log_int(rng, 1 << 12, 1 << 21), "deg": round(rng.uniform(2, 8), 2),
                "cls": rng.choice([1, 3, 4, 5, 7]), "r": rng.randint(5, 10)}
    if kind == "batch":
        return {"kind": "batch", "G": _log_int(rng, 32, 512), "n_lo": 100, "n_hi": _log_int(rng, 1000, 100000),
                "r": rng.randint(10, 20)}
    if kind == "served":
        return {"kind": "served", "pool": rng.randint(8, 24), "requests": rng.randint(16, 48), "n_lo": 1000,
                "n_hi": _log_int(rng, 10000, 1000000)}
    if kind == "es":
        n = _log_int(rng, 1 << 10, 1 << 20)
        return {"kind": "es", "n": n, "gamma": round(rng.uniform(2.1, 3.0), 3), "dmin": rng.randint(2, 5),
                "dmax": max(8, min(1024, math.isqrt(n))), "share": round(rng.uniform(0.1, 0.5), 3)}
    if kind == "mixing":
        return {"kind": "mixing", "n": _log_int(rng, 1 << 9, 1 << 13), "gamma": round(rng.uniform(2.15, 2.8), 3),
                "K": rng.randint(40, 200), "chain": rng.choice([gesmc.CHAIN_GLOBAL, gesmc.CHAIN_ES])}
    if rng.random() < 0.5:
        return {"kind": "gen", "graph": "gnp", "n": _log_int(rng, 1000, 1 << 22), "deg": round(rng.uniform(4, 32), 2)}
    n = _log_int(rng, 1000, 1 << 20)
    return {"kind": "gen", "graph": "pld", "n": n, "gamma": round(rng.uniform(2.1, 3.0), 3), "dmin": rng.randint(1, 5),
            "dmax": max(8, min(1024, math.isqrt(n)))}


# ---- inputs ---------------------------------------------------------------
# The sizes (edge counts, degree sequences, the mix of a batch) belong to the
# case, so that every seed gives arrays of the same shape; which edges there
# are, the vertex labels and every random choice of the chain follow the seed.
_RECIPE = 2  # seed of the degree sequences


def _gnp_edges(case):
    n = case["n"]
    return min(n * (n - 1) // 2, int(n * case["deg"] * 0.5))


def _gnp(ctx, case, seed):
    """m edges of G(n, p), in pair order: p a little above m / N, what is too much dropped at random."""
    n, m = case["n"], _gnp_edges(case)
    e = ctx.gen_gnp(n, min(1.0, (m + 8.0 * math.sqrt(m) + 8.0) / (n * (n - 1) / 2)), seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    drop = torch.randperm(e.numel(), device="cuda", generator=g)[: e.numel() - m]
    keep = torch.ones(e.numel(), dtype=torch.bool, device="cuda")
    keep[drop] = False
    return e[keep].contiguous()


def _pld(ctx, n, gamma, dmin, dmax, seed, recipe=_RECIPE):
    """Havel-Hakimi of Pld([dmin..dmax], gamma) degrees, relabelled by the seed."""
    deg, _ = ctx.gen_pld_degrees(n, gamma, dmin, dmax, recipe)
    return ctx.gen_relabel(ctx.gen_havel_hakimi(deg), n, seed)


def _graph(ctx, case, seed):
    if case.get("graph", "pld") == "gnp":
        return _gnp(ctx, case, seed)
    return _pld(ctx, case["n"], case["gamma"], case["dmin"], case["dmax"], seed)


def _uneven(case, G):
    """n and gamma of G graphs: n log-uniform, gamma uniform in [2.1, 3.0], degrees in [2, sqrt(n)]."""
    rng = random.Random(_RECIPE)
    return [(_log_int(rng, case["n_lo"], case["n_hi"]), rng.uniform(2.1, 3.0)) for _ in range(G)]


def _class_graph(case, seed):
    """Uniform endpoints; loops and repeated edges only where the class allows them."""
    n, cls = case["n"], case["cls"]
    m = int(n * case["deg"])
    more = m + m // 50 + 1000
    g = torch.Generator(device="cuda").manual_seed(seed)
    u, v = (torch.randint(0, n, (more,), device="cuda", generator=g) for _ in range(2))
    if not cls & gesmc.CLASS_LOOPS:
        keep = u != v
        u, v = u[keep], v[keep]
    if not cls & gesmc.CLASS_DIRECTED:
        u, v = torch.minimum(u, v), torch.maximum(u, v)
    keys = (u << 32) | v
    if not cls & gesmc.CLASS_MULTI:
        keys = torch.unique(keys)
        keys = keys[torch.randperm(keys.numel(), device="cuda", generator=g)]
    return keys[:m].contiguous()


def _mixing_dmax(case):
    return int(case["n"] ** (1.0 / (case["gamma"] - 1.0)))


def prepare(case, seed):
    ctx = gesmc.Context(0)
    kind, s = case["kind"], {"case": case, "ctx": ctx, "seed": seed * 1000003 + 17}
    if kind == "run":
        s["edges"] = _graph(ctx, case, seed)
    elif kind == "class":
        s["edges"] = _class_graph(case, seed)
    elif kind == "es":
        s["edges"] = _graph(ctx, case, seed)
        s["r"] = max(1, int(s["edges"].numel() * case["share"]))
    elif kind == "mixing":
        s["edges"] = _pld(ctx, case["n"], case["gamma"], 1, _mixing_dmax(case), seed)
    elif kind == "batch":
        specs = _uneven(case, case["G"])
        graphs = [_pld(ctx, n, g, 2, math.isqrt(n), seed + q, q) for q, (n, g) in enumerate(specs)]
        s["edges"] = torch.cat(graphs)
        s["offsets"] = np.concatenate([[0], np.cumsum([e.numel() for e in graphs])]).tolist()
        s["n"] = [n for n, _ in specs]
        s["seeds"] = [s["seed"] + q for q in range(case["G"])]
        s["r"] = [case["r"]] * case["G"]
    elif kind == "served":
        pool = []
        for q, (n, g) in enumerate(_uneven(case, case["pool"])):
            pool.append((_pld(ctx, n, g, 2, math.isqrt(n), seed + q, q).cpu().numpy().view(np.uint64), n))
        s["requests"] = [pool[k] + (s["seed"] + q, r) for q, (k, r) in enumerate(_requests(case))]
        s["server"] = gesmc.Server(ctx, hbm_budget_bytes=16 << 30)
    elif case["graph"] == "pld":
        # the prescribed degrees, in an order of the seed's own
        deg, _ = ctx.gen_pld_degrees(case["n"], case["gamma"], case["dmin"], case["dmax"], _RECIPE)
        g = torch.Generator(device="cuda").manual_seed(seed)
        s["deg"] = deg[torch.randperm(case["n"], device="cuda", generator=g)].contiguous()
    else:
        s["out"] = torch.zeros(int(_gnp_edges(case) + 8.0 * math.sqrt(_gnp_edges(case)) + 8), dtype=torch.int64,
                               device="cuda")
    return s


def _requests(case):
    """Graph of the pool and r of each request: r uniform in 10..50."""
    rng = random.Random(_RECIPE + 1)
    return [(rng.randrange(case["pool"]), rng.randint(10, 50)) for _ in range(case["requests"])]


def _counts(st):
    return [st[k] for k in _COUNTS if k in st]


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "run":
        out, st = ctx.run(s["edges"], case["n"], s["seed"], 0, case["r"], case["pl"])
        return {"edges": out, "counts": _counts(st)}
    if kind == "class":
        out, st, _, codes = ctx.run_class(s["edges"], case["n"], s["seed"], case["cls"], 0, case["r"], outcomes=True)
        return {"edges": out, "counts": _counts(st), "codes": codes}
    if kind == "batch":
        out, per_graph, total = ctx.run_batch(s["edges"], s["offsets"], s["n"], s["seeds"], s["r"])
        return {"edges": out, "counts": np.array([_counts(g) for g in per_graph], dtype=np.int64),
                "total": _counts(total)}
    if kind == "served":
        srv = s["server"]
        tickets = [srv.submit(e, n, seed, r) for e, n, seed, r in s["requests"]]
        res = [srv.wait(t) for t in tickets]
        return {"edges": [x["edges"].view(np.int64) for x in res],
                "counts": np.array([[x["status"]] + _counts(x["stats"]) for x in res], dtype=np.int64)}
    if kind == "es":
        out, st, codes = ctx.run_es(s["edges"], case["n"], s["seed"], 0, s["r"], outcomes=True)
        return {"edges": out, "counts": _counts(st), "codes": codes}
    if kind == "mixing":
        res, _ = ctx.mixing(s["edges"], case["n"], s["seed"], case["K"], _THIN, chain=case["chain"])
        return {"table": np.array([[x[k] for k in sorted(x)] for x in res], dtype=np.int64)}
    if case["graph"] == "pld":
        return {"edges": ctx.gen_relabel(ctx.gen_havel_hakimi(s["deg"]), case["n"], s["seed"])}
    got = ctx.gen_gnp(case["n"], min(1.0, case["deg"] / (case["n"] - 1)), s["seed"], out=s["out"])
    return {"edges": s["out"], "m": got.numel()}


# ---- the least work -------------------------------------------------------
def _pld_mean(gamma, dmin, dmax):
    w = [d ** -gamma for d in range(dmin, dmax + 1)]
    return sum(d * x for d, x in zip(range(dmin, dmax + 1), w)) / sum(w)


def _expected_edges(case):
    if "deg" in case:
        return case["n"] * case["deg"] * (1.0 if case["kind"] == "class" else 0.5)
    dmin, dmax = case.get("dmin", 1), case.get("dmax") or _mixing_dmax(case)
    return 0.5 * case["n"] * _pld_mean(case["gamma"], dmin, dmax)


def work(case):
    """Bytes that a pass cannot do without; the path has no floating-point operations to count.

    A superstep switches every edge: 8 bytes read and 8 written per edge.  A
    switch of the switch-by-switch chain reads and writes two edges, looks two
    targets up and leaves an outcome code.  Loading and handing back the edges
    comes on top.
    """
    kind = case["kind"]
    if kind in ("batch", "served"):
        m = [0.5 * n * _pld_mean(g, 2, math.isqrt(n)) for n, g in _uneven(case, case["G" if kind == "batch" else "pool"])]
        if kind == "batch":
            return {"bytes": 16.0 * sum(m) * (case["r"] + 1), "flops": 0.0}
        return {"bytes": sum(16.0 * m[k] * (r + 1) for k, r in _requests(case)), "flops": 0.0}
    m = _expected_edges(case)
    if kind == "es":
        return {"bytes": 16.0 * m + 49.0 * m * case["share"], "flops": 0.0}
    if kind == "mixing":
        r = case["K"]
        return {"bytes": 16.0 * m * r * (1 if case["chain"] == gesmc.CHAIN_GLOBAL else 1.5), "flops": 0.0}
    if kind == "gen":
        # the edges written once; a degree read and a label looked up per vertex
        return {"bytes": 8.0 * m + (8.0 * case["n"] if case["graph"] == "pld" else 0.0), "flops": 0.0}
    return {"bytes": 16.0 * m * (case["r"] + 1), "flops": 0.0}
