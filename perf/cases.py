"""The work that a program does with this library, as cases to time.

Every case names one entry point (`call`), a seeded graph (`graph`, `n`), the
table layout it is loaded in, and the walk counts of Algorithm 1 as fixed
numbers: B probes in each of G = 37 blocks (delta = 0.01), R replicas, two
walks of L steps. The walk counts are those that the calibrated and throughput
budgets of this repository give at the median. A graph depends on (graph, n)
only and stays loaded, as in a program that serves queries on it; the pairs,
the Philox key and the query ids come from the seed. `load` makes its graph
from the seed too, since loading is what it measures.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2512_05460_amd import binding as bd

G_BLOCKS = 37  # ceil(8 ln(1/0.01))
LAYOUTS = {
    "csr": bd.BD_LAYOUT_CSR,
    "auto": bd.BD_LAYOUT_AUTO,
    "fat": bd.BD_LAYOUT_FAT,
    "compact": bd.BD_LAYOUT_COMPACT,
    "storage": bd.BD_LAYOUT_COMPACT | bd.BD_RELABEL_DEGREE | bd.BD_PROBE_STORAGE_IDS,
}
MOST_STEPS = 18_000_000_000   # walk steps of the largest case
EXACT_STEPS = 10_000_000_000  # beyond this many scored steps the 64-bit replay takes too long
WIDEST_N = 10_000_000


# --------------------------------------------------------------------------- #
# The cases
# --------------------------------------------------------------------------- #
def listed():
    return [
        # one pair asked interactively on a small graph: launches, copies and step latency
        {"name": "one small query", "call": "batch", "graph": "power3", "n": 1_000, "layout": "compact",
         "mode": "plain", "nq": 1, "B": 2, "R": 64, "L": 50, "share": 1},
        # an all-pairs style study of a small network (eps = 0.1, L = 200), one replayed hipGraph
        {"name": "small graph batch", "call": "batch", "graph": "power3", "n": 1_000, "layout": "compact",
         "mode": "graph", "nq": 32, "B": 96, "R": 176, "L": 200, "share": 1},
        # the benchmark's headline: one query at eps = 0.05, L = 1000 on the fastest layout
        {"name": "headline query", "call": "batch", "graph": "power", "n": 100_000, "layout": "storage",
         "mode": "plain", "nq": 1, "B": 256, "R": 934, "L": 1_000, "share": 1},
        # a batch on the layout that the library picks, caller ids kept
        {"name": "automatic layout batch", "call": "batch", "graph": "power", "n": 100_000, "layout": "auto",
         "mode": "batched", "nq": 17, "B": 64, "R": 234, "L": 499, "share": 1},
        # road-like graph, many cheap queries of mixed length in one replayed launch
        {"name": "grid mixed lengths", "call": "batch", "graph": "grid", "n": 1_999_396, "layout": "auto",
         "mode": "graph", "nq": 1_024, "B": 3, "R": 12, "L": 5_000, "share": 1},
        # continuous batching on a graph far larger than the caches, requests of 1 to 512 pairs
        {"name": "served requests", "call": "serve", "graph": "power", "n": WIDEST_N, "layout": "auto",
         "requests": 10, "largest": 512, "B": 16, "R": 3, "L": 1_000},
        # walk sharing, the repository's extension of the algorithm
        {"name": "shared walks", "call": "batch", "graph": "power", "n": 100_000, "layout": "storage",
         "mode": "plain", "nq": 1, "B": 384, "R": 321, "L": 1_000, "share": 4},
        # the length chosen by the stabilization rule, on the default layout
        {"name": "stabilized lengths", "call": "stabilized", "graph": "power", "n": 100_000, "layout": "csr",
         "nq": 16, "B": 16, "R": 100, "L": 256, "eps": 0.1},
        # the deterministic reference of a few pairs on a small graph
        {"name": "series of a few pairs", "call": "series", "graph": "power3", "n": 1_000, "layout": "compact",
         "nq": 3, "L": 200},
        # the deterministic reference of a full block of pairs
        {"name": "series of 64 pairs", "call": "series", "graph": "power", "n": 100_000, "layout": "auto",
         "nq": 64, "L": 400},
        # the mixing factor, from which Theorem 3.8 takes the walk length
        {"name": "mixing factor", "call": "lambda", "graph": "power", "n": 100_000, "layout": "csr", "L": 300},
        # a program's start: check and lay out a graph from host arrays, answer a first query
        {"name": "load and first query", "call": "load", "graph": "power", "n": 100_000, "layout": "auto",
         "mode": "batched", "nq": 1, "B": 4, "R": 64, "L": 100, "share": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(("batch", "batch", "batch", "batch", "serve", "stabilized", "series", "lambda", "load"))
    graph = rng.choice(("power", "power", "power3", "grid"))
    c = {"call": call, "graph": graph}
    if call == "batch":
        c["n"] = _log_int(rng, 1_000, WIDEST_N if graph == "power" else 2_000_000)
        c["layout"] = rng.choice(("auto", "auto", "storage", "csr", "fat", "compact"))
        c["mode"] = rng.choice(("plain", "batched", "graph"))
        c["share"] = rng.choice((1, 1, 1, 2, 4))
        c["L"] = _log_int(rng, 20, 5_000)
        c["R"] = _log_int(rng, 2, 1_000)
        c["B"] = _log_int(rng, 2, 256)
        c["nq"] = _log_int(rng, 1, 64 if c["mode"] == "plain" else 1_024)
        return _fit(c)
    if call == "serve":
        c |= {"n": _log_int(rng, 10_000, WIDEST_N if graph == "power" else 2_000_000), "layout": "auto",
              "requests": rng.randint(2, 12), "largest": _log_int(rng, 4, 512), "B": _log_int(rng, 2, 32),
              "R": _log_int(rng, 2, 64), "L": _log_int(rng, 100, 2_000)}
        return _fit(c)
    if call == "stabilized":
        c |= {"n": _log_int(rng, 1_000, 1_000_000), "layout": rng.choice(("csr", "auto")), "nq": rng.randint(1, 48),
              "B": _log_int(rng, 2, 32), "R": _log_int(rng, 8, 200), "L": _log_int(rng, 16, 512), "eps": 0.1}
        return _fit(c)
    if call == "series":
        c |= {"n": _log_int(rng, 1_000, 150_000), "layout": rng.choice(("csr", "auto", "fat")),
              "nq": rng.randint(1, 80)}
        c["L"] = min(_log_int(rng, 20, 2_000), max(20, 2_560_000_000 // (c["n"] * max(c["nq"], 8))))
        return c
    if call == "lambda":
        c |= {"n": _log_int(rng, 1_000, 400_000), "layout": "csr", "L": _log_int(rng, 50, 400)}
        return c
    c |= {"n": _log_int(rng, 2_000, 200_000), "layout": rng.choice(("auto", "storage", "fat", "csr")),
          "mode": "batched", "nq": _log_int(rng, 1, 16), "B": 4, "R": _log_int(rng, 8, 64),
          "L": _log_int(rng, 20, 200), "share": 1}
    return c


def _fit(c):
    """The case with fewer probes, replicas or pairs until it is within the largest one's work."""
    most = MOST_STEPS // (4 if c["layout"] in ("csr", "fat") or c["n"] > 150_000 else 2)
    for key, least in (("B", 2), ("nq", 1), ("largest", 4), ("R", 2)):
        while key in c and _steps(c) > most and c[key] > least:
            c[key] = max(least, c[key] // 2)
    return c


def _sizes(c):
    """Pairs of each request of a served case: powers of two up to the largest."""
    top = c["largest"].bit_length() - 1
    return [min(c["largest"], 1 << ((3 * i) % (top + 1))) for i in range(c["requests"])]


def _pairs(c):
    return sum(_sizes(c)) if c["call"] == "serve" else c.get("nq", 0)


def _steps(c):
    """Walk steps of one pass."""
    groups = G_BLOCKS * -(-c["B"] // c.get("share", 1))
    L = c["L"]
    if c["call"] == "stabilized":
        L = 1.5 * L  # the rule tries 1, 2, 4, ... and most pairs stop before the last
    if c["graph"] == "grid" and c["call"] == "batch":
        L = 0.5 * L  # the lengths are mixed
    return int(_pairs(c) * groups * c["R"] * 2 * L)


# --------------------------------------------------------------------------- #
# Graphs
# --------------------------------------------------------------------------- #
def _csr_of(n, u, v):
    """Canonical CSR (symmetric, simple, sorted rows) of the edges u-v, on the GPU."""
    ok = u != v
    u, v = u[ok], v[ok]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    rows = key // n
    rp = torch.zeros(n + 1, dtype=torch.int64, device=key.device)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rp, (key - rows * n).to(torch.int32)


def _power_law(n, mean, exponent, seed):
    """Connected power-law graph: node of rank i has weight ~ (i + 1)^(-1/(exponent - 1)),
    capped as in the Chung-Lu model; each rank is joined to a lower one and the
    remaining edges join two ranks, all drawn by weight; ids are shuffled."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.arange(1, n + 1, dtype=torch.float64, device="cuda") ** (-1.0 / (exponent - 1.0))
    w *= mean * n / w.sum()
    w = torch.minimum(w, w.sum().sqrt())
    cdf = torch.cumsum(w, 0)

    def by_weight(r):
        return torch.searchsorted(cdf, r, right=True).clamp_(max=n - 1)

    def uniform(m):
        return torch.rand(m, dtype=torch.float64, device="cuda", generator=gen)

    child = torch.arange(1, n, device="cuda")
    parent = torch.minimum(by_weight(uniform(n - 1) * cdf[:-1]), child - 1)
    m = int(n * mean / 2) - (n - 1)
    u = torch.cat([child, by_weight(uniform(m) * cdf[-1])])
    v = torch.cat([parent, by_weight(uniform(m) * cdf[-1])])
    ids = torch.randperm(n, device="cuda", generator=gen)
    return _csr_of(n, ids[u], ids[v])


def _grid(n, seed):
    """side x side grid without one in ten of its vertical edges (the first column keeps all of its own)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    side = math.isqrt(n)
    at = torch.arange(side * side, device="cuda").reshape(side, side)
    keep = torch.rand(side - 1, side, device="cuda", generator=gen) >= 0.1
    keep[:, 0] = True
    u = torch.cat([at[:, :-1].reshape(-1), at[:-1][keep]])
    v = torch.cat([at[:, 1:].reshape(-1), at[1:][keep]])
    return _csr_of(side * side, u, v)


def _graph(c, seed):
    """(n, row_ptr, col) on the GPU."""
    if c["graph"] == "grid":
        rp, col = _grid(c["n"], seed)
    elif c["graph"] == "power3":
        rp, col = _power_law(c["n"], 6.0, 3.0, seed)
    else:
        rp, col = _power_law(c["n"], 10.0, 2.5, seed)
    return rp.numel() - 1, rp, col


@functools.lru_cache(maxsize=2)
def _loaded(graph, n, layout):
    n, rp, col = _graph({"graph": graph, "n": n}, n)
    flags = LAYOUTS[layout] | (bd.BD_SKIP_VALIDATION if n > 1_000_000 else 0)
    return bd.graph_load_csr_device(n, rp, col, flags)


# --------------------------------------------------------------------------- #
# One pass
# --------------------------------------------------------------------------- #
def _queries(c, seed, n):
    rng = np.random.default_rng(seed)
    m = _pairs(c)
    s = rng.integers(0, n, m)
    t = rng.integers(0, n - 1, m)
    t += t >= s
    L = np.full(m, c["L"])
    if c["graph"] == "grid" and c["call"] == "batch":  # three lengths, a tenth, two fifths and all of L, in turn
        L = np.maximum(1, np.array([c["L"] // 10, 2 * c["L"] // 5, c["L"]])[np.arange(m) % 3])
    return {"s": s.astype(np.int32), "t": t.astype(np.int32), "L": L.astype(np.int32),
            "uid": rng.permutation(1 << 20)[:m].astype(np.uint32), "key": int(rng.integers(1 << 62)),
            "eps": c.get("eps", 0.1)}


def _policy(c):
    return bd.policy("fixed", B=c["B"], R=c["R"], share=c.get("share", 1))


def prepare(case, seed):
    c = dict(case)
    if c["call"] == "load":
        n, rp, col = _graph(c, seed)
        return {"case": c, "n": n, "row_ptr": rp.cpu().numpy(), "col": col.cpu().numpy(), "policy": _policy(c),
                "exec": bd.exec_cfg("batched"), "q": _queries(c, seed, n)}
    g = _loaded(c["graph"], c["n"], c["layout"])
    state = {"case": c, "graph": g}
    if c["call"] == "lambda":
        state["seed"] = int(seed)
        return state
    state["q"] = _queries(c, seed, g.info()["n"])
    if c["call"] == "series":
        return state
    state["policy"] = _policy(c)
    if c["call"] == "serve":
        state["server"] = bd.Server(g, state["policy"], max_queries=4096)
    else:
        mode = c.get("mode", "batched")
        state["exec"] = bd.exec_cfg("plain" if mode == "plain" else "batched", use_graph=mode == "graph")
    return state


def _answers(r):
    return {"beta": r["beta"], "status": r["status"], "walk_steps": r["walk_steps"]}


def run(state):
    c = state["case"]
    q = state.get("q")
    if c["call"] == "batch":
        return _answers(bd.bd_query_batch(state["graph"], q["s"], q["t"], q["eps"], q["L"], q["key"], state["policy"],
                                          state["exec"], uid=q["uid"]))
    if c["call"] == "serve":
        srv, ids, at = state["server"], [], 0
        for m in _sizes(c):
            part = slice(at, at + m)
            ids.append(srv.submit(q["s"][part], q["t"][part], q["eps"], q["L"][part], q["key"], uid=q["uid"][part]))
            at += m
        return _answers(np.concatenate([srv.wait(i)[0] for i in ids]))
    if c["call"] == "stabilized":
        r, stop = bd.bd_query_stabilized(state["graph"], q["s"], q["t"], q["eps"], c["L"], q["key"], state["policy"],
                                         state["exec"], uid=q["uid"])
        return {**_answers(r), "L": stop}
    if c["call"] == "series":
        return {"beta": bd.bd_truncated_beta(state["graph"], q["s"], q["t"], c["L"])}
    if c["call"] == "lambda":
        return {"lambda": bd.bd_graph_lambda(state["graph"], c["L"], state["seed"])}
    g = bd.graph_load_csr(state["n"], state["row_ptr"], state["col"], LAYOUTS[c["layout"]])
    info = g.info()
    r = bd.bd_query_batch(g, q["s"], q["t"], q["eps"], q["L"], q["key"], state["policy"], state["exec"], uid=q["uid"])
    g.free()
    return {**_answers(r), **{k: info[k] for k in ("n", "nnz", "d_min", "d_max", "bipartite", "layout")}}


def work(case):
    """Bytes: the graph as CSR (4 bytes an offset and an id), the queries and the
    results, once each. Operations of a walk step: Philox4x32-10 (80 per four
    steps), six Feistel rounds (36), the sign hash (8), the draw of the
    neighbour and the sum (11); of a product with P: a multiply and an add per
    entry and column."""
    c = dict(case)
    mean = {"power": 10, "power3": 6, "grid": 3.9}[c["graph"]]
    graph = 4 * (c["n"] + 1) + 4 * mean * c["n"]
    if c["call"] == "lambda":
        return {"bytes": graph + 8, "flops": 2.0 * c["L"] * c["n"] * (mean + 3)}
    if c["call"] == "series":
        return {"bytes": graph + 16 * c["nq"], "flops": 2.0 * c["L"] * c["nq"] * c["n"] * (mean + 1)}
    per_step = 31 + 44 * c.get("share", 1)
    return {"bytes": graph + 76 * _pairs(c), "flops": float(per_step * _steps(c))}


# --------------------------------------------------------------------------- #
# The same in 64 bits, in plain torch
# --------------------------------------------------------------------------- #
M32 = 0xFFFFFFFF
HASH_P = 2 ** 31 - 1


def _philox(c0, c1, c2, c3, key):
    k0, k1 = key & M32, (key >> 32) & M32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32)
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _probe_keys(k, uid, key, n):
    def words(i):
        return _philox(torch.full_like(k, i), M32, k, uid << 1, key)
    w0, w1, w2 = words(0), words(1), words(2)
    r = torch.full_like(k, 1) if n & 1 else 2 * (w2[0] & 1)
    return [*w0, w1[0], w1[1]], 1 + w1[2] % (HASH_P - 1), w1[3] % HASH_P, n - r


def _signs(x, pick, keys, n):
    """z^(k) of the nodes x for the probes `pick` of `keys`."""
    K, a, b, zlo = keys
    bits = max(1, (n - 1).bit_length())
    rb = bits >> 1
    mask = (1 << rb) - 1
    A = (n + mask) >> rb

    def mix(v, k):
        h = (((v ^ k) & 0xFFFFFF) * 0x9E3779) & M32
        h = h ^ (h >> 15)
        return ((h & 0xFFFFFF) * 0x873593) & M32

    def turn(x, ks):
        hi, lo = x >> rb, x & mask
        for r in range(0, 6, 2):
            t = hi + (((mix(lo, ks[r]) >> 8) * (A << 8)) >> 32)
            hi = torch.where(t >= A, t - A, t)
            lo = lo ^ ((mix(hi, ks[r + 1]) >> (32 - rb if rb else 31)) & mask)
        return (hi << rb) | lo

    y = turn(x, [k[pick] for k in K])
    while True:
        again = (y >= n).nonzero(as_tuple=True)[0]
        if not again.numel():
            break
        y[again] = turn(y[again], [k[pick[again]] for k in K])
    neg = (((a[pick] * (y >> 1) + b[pick]) % HASH_P) & 1) ^ (y & 1)
    return torch.where(y >= zlo[pick], 0, 1 - 2 * neg)


def _estimate(csr, s, t, L, B, R, share, uid, key):
    """beta-hat of one pair by the stated walks, with binary64 sums."""
    n, rp, col = csr
    deg = rp[1:] - rp[:-1]
    per_block = -(-B // share)
    first = torch.arange(G_BLOCKS * per_block, device=rp.device)
    first = first // per_block * B + first % per_block * share  # first probe of each group
    keys = _probe_keys(torch.arange(G_BLOCKS * B, device=rp.device), uid, key, n)
    q = torch.zeros(G_BLOCKS * B, dtype=torch.float64, device=rp.device)
    many = max(1, 4_000_000 // R)
    for g0 in range(0, first.numel(), many):
        k = first[g0:g0 + many].repeat_interleave(R)
        p = torch.arange(R, device=rp.device).repeat(k.numel() // R)
        x = torch.cat([torch.full_like(k, s), torch.full_like(k, t)])
        side = torch.cat([torch.zeros_like(k), torch.ones_like(k)])
        kk, pp = k.repeat(2), p.repeat(2)
        probes = [torch.where(kk % B + j < B, kk + j, kk) for j in range(share)]
        sums = [torch.zeros(kk.numel(), dtype=torch.float64, device=rp.device) for _ in range(share)]
        for step in range(L + 1):
            for j in range(share):
                sums[j] += _signs(x, probes[j], keys, n) / deg[x].double()
            if step == L:
                break
            if step % 4 == 0:
                words = _philox(torch.full_like(kk, step // 4), pp, kk, (uid << 1) | side, key)
            x = col[rp[x] + ((words[step % 4] * deg[x]) >> 32)].long()
        for j in range(share):
            U = (sums[j][:k.numel()] - sums[j][k.numel():]).reshape(-1, R)
            s1, s2 = U.sum(1), (U * U).sum(1)
            kf = first[g0:g0 + many]
            inside = kf % B + j < B
            q[(kf + j)[inside]] = ((s1 * s1 - s2) / (R * (R - 1)))[inside]
    return float(np.median(q.reshape(G_BLOCKS, B).mean(1).cpu().numpy()))


def _by_degree(csr):
    """The graph with its nodes in descending degree (ties by id), rows in the given order; and each id's new one."""
    n, rp, col = csr
    deg = rp[1:] - rp[:-1]
    order = torch.argsort(-deg, stable=True)
    new = torch.empty_like(order)
    new[order] = torch.arange(n, device=rp.device)
    d = deg[order]
    rp2 = torch.zeros_like(rp)
    rp2[1:] = torch.cumsum(d, 0)
    src = torch.repeat_interleave(rp[:-1][order] - rp2[:-1], d) + torch.arange(col.numel(), device=rp.device)
    return (n, rp2, new[col[src].long()].to(torch.int32)), new


def _sparse(csr):
    n, rp, col = csr
    return torch.sparse_csr_tensor(rp, col.long(), torch.ones(col.numel(), dtype=torch.float64, device=rp.device), (n, n))


def _series(csr, q, L):
    n, rp, col = csr
    deg = (rp[1:] - rp[:-1]).double()[:, None]
    s, t = (torch.from_numpy(q[k]).long().to(rp.device) for k in ("s", "t"))
    v = torch.zeros(n, s.numel(), dtype=torch.float64, device=rp.device)
    at = torch.arange(s.numel(), device=rp.device)
    v[s, at] = 1.0 / deg[s, 0]
    v[t, at] = -1.0 / deg[t, 0]
    A, h = _sparse(csr), v.clone()
    for _ in range(L):
        v = (A @ v) / deg
        h += v
    return ((h * h).sum(0) - h.sum(0) ** 2 / n).cpu().numpy()


def _lambda(csr, iters, seed):
    n, rp, col = csr
    deg = (rp[1:] - rp[:-1]).double()
    phi = (deg / col.numel()).sqrt()

    def signed(v):
        return v - (1 << 64) if v >> 63 else v

    z = seed + (torch.arange(1, n + 1, device=rp.device)) * signed(0x9E3779B97F4A7C15)
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * signed(0x94D049BB133111EB)
    z = z ^ ((z >> 31) & ((1 << 33) - 1))
    x = ((z >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53 - 0.5
    A, size = _sparse(csr), 0.0
    for i in range(iters + 1):
        y = x if i == 0 else (A @ (x / deg.sqrt())[:, None])[:, 0] / deg.sqrt()
        y = y - (phi @ y) * phi
        size = y.norm()
        x = y / size
    return float(size)


def exact(case, seed):
    c = dict(case)
    if c["call"] in ("batch", "serve", "stabilized", "load") and _steps(c) * c.get("share", 1) > EXACT_STEPS:
        return None
    if _pairs(c) * c["L"] > 10_000 and c["call"] != "series":
        return None  # a step of each pair is some hundred launches
    csr = _graph(c, seed if c["call"] == "load" else c["n"])
    if c["call"] == "lambda":
        return {"lambda": _lambda(csr, c["L"], int(seed))}
    q = _queries(c, seed, csr[0])
    if c["call"] == "series":
        return {"beta": _series(csr, q, c["L"])}
    s, t = q["s"], q["t"]
    if c["layout"] == "storage":
        csr, new = _by_degree(csr)
        s, t = (new[torch.from_numpy(v).long().to(new.device)].cpu().numpy() for v in (s, t))

    def one(i, L):
        return _estimate(csr, int(s[i]), int(t[i]), int(L), c["B"], c["R"], c.get("share", 1), int(q["uid"][i]), q["key"])

    if c["call"] != "stabilized":
        return {"beta": np.array([one(i, q["L"][i]) for i in range(len(s))])}
    beta = np.empty(len(s))
    for i in range(len(s)):
        L, now = 1, one(i, 1)
        while L < c["L"]:
            L, last = min(2 * L, c["L"]), now
            now = one(i, L)
            if abs(now - last) <= 0.5 * q["eps"] * abs(now):
                break
        beta[i] = now
    return {"beta": beta}
