"""The calls whose speed matters to a program that counts triangles with this package, over the
range of sizes it meets: one small graph at a time, ordinary graphs, the largest benchmark
graph, prepared graphs counted again, per-vertex counts, batches of many small graphs and the
serving loop's packed requests.

A case is a dict of plain values.  `kind` names the call:
  count       edges -> total, workspace and result buffers from the call itself (api.count_async;
              `blocking`: api.count, which returns the number)
  step        tc_preprocess + tc_count_prepared into a workspace the program keeps (api.Prepared)
  resident    a count of a graph prepared once (api.Prepared.count_async)
  per_vertex  edges -> total and the count of every vertex
  batch       many graphs in the batched format (a captured plan, or the one-shot call)
  serve       edge arrays of several requests packed and counted together, as the serving loop does
Graphs have exactly n vertices and m undirected edges; `both` lists every edge in both directions.
"""
import math

import torch

from paper_1503_00576_amd import api

DEV = "cuda:0"

# R-MAT quadrant probabilities of the package's own generator
A, B, C = 0.57, 0.19, 0.19


def listed():
    return [
        # one small graph, the caller waits for the number: G(1000, p) with p near 0.02
        {"name": "count_er_1000", "kind": "count", "family": "er", "n": 1000, "m": 9704,
         "both": False, "blocking": True},
        # a small request of ragged size, as an interactive program sends them one by one
        {"name": "count_rmat13_ragged", "kind": "count", "family": "rmat", "n": 8009, "m": 100003,
         "both": False, "blocking": False},
        # an ordinary graph in the two-direction edge format of adjacency dumps
        {"name": "count_both_rmat18", "kind": "count", "family": "rmat", "n": 200003,
         "m": 3000001, "both": True, "blocking": False},
        # an ordinary graph without hubs: the small-world family, degree 16 everywhere
        {"name": "count_ws_1m", "kind": "count", "family": "ws", "n": 1000003, "m": 8000024,
         "both": False, "blocking": False},
        # the middle of the benchmark range: R-MAT scale 20, edge factor 16
        {"name": "count_rmat20", "kind": "count", "family": "rmat", "n": 1 << 20, "m": 15700000,
         "both": False, "blocking": False},
        # the largest: R-MAT scale 23, edge factor 24, as bench.py steps it
        {"name": "step_rmat23", "kind": "step", "family": "rmat", "n": 1 << 23, "m": 191864605,
         "both": False},
        # a graph kept resident by a serving program and counted again
        {"name": "resident_rmat21", "kind": "resident", "family": "rmat", "n": 1 << 21,
         "m": 32000000, "both": False},
        # clustering coefficients of a medium graph of ragged size, by preferential attachment
        {"name": "pv_ba_100k", "kind": "per_vertex", "family": "ba", "n": 100003, "m": 1200000,
         "both": False},
        # clustering coefficients of a large graph
        {"name": "pv_rmat22", "kind": "per_vertex", "family": "rmat", "n": 1 << 22, "m": 64000000,
         "both": False},
        # the many-small-graphs workload: 4096 graphs through a captured plan (the tuning is the
        # autotuner's choice on this batch)
        {"name": "batch_4096", "kind": "batch", "graphs": 4096, "n_min": 50, "n_max": 20000,
         "deg_min": 4.0, "deg_max": 32.0, "per_vertex": False, "plan": True},
        # a smaller batch, counted once, with per-vertex counts
        {"name": "batch_pv_300", "kind": "batch", "graphs": 300, "n_min": 50, "n_max": 20000,
         "deg_min": 4.0, "deg_max": 32.0, "per_vertex": True, "plan": False},
        # what the serving loop launches when a few small requests wait
        {"name": "serve_pack_4", "kind": "serve", "graphs": 4, "scale_min": 10, "scale_max": 14,
         "ef": 10.5},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count", "count", "count", "step", "resident", "per_vertex", "per_vertex",
                       "batch", "batch", "serve"])
    if kind == "batch":
        plan = rng.random() < 0.5
        pv = rng.random() < 0.4
        return {"kind": kind, "graphs": _log_uniform(rng, 8, 1500 if pv else 4000),
                "n_min": 50, "n_max": _log_uniform(rng, 400, 20000), "deg_min": 4.0,
                "deg_max": round(rng.uniform(8.0, 32.0), 2), "per_vertex": pv, "plan": plan}
    if kind == "serve":
        lo = rng.randint(10, 13)
        return {"kind": kind, "graphs": _log_uniform(rng, 1, 64), "scale_min": lo,
                "scale_max": rng.randint(lo, 14), "ef": round(rng.uniform(6.0, 10.5), 2)}
    family = rng.choice(["rmat", "rmat", "rmat", "er", "ws", "ba"])
    m = _log_uniform(rng, 5000, {"count": 4e7, "step": 1e8, "resident": 6e7,
                                 "per_vertex": 4e7}[kind])
    n = max(700, int(m / rng.uniform(7.0, 23.0))) | 1
    if family == "rmat":
        m = min(m, int(n * 0.8 * math.log2(n)))  # what R-MAT draws without many repeats
    case = {"kind": kind, "family": family, "n": n, "m": m,
            "both": kind in ("count", "per_vertex") and rng.random() < 0.3}
    if kind == "count":
        case["blocking"] = m < 200000 and rng.random() < 0.5
    return case


# ------------------------------------------------------------------ inputs


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _rand(k, g):
    return torch.rand(k, generator=g, device=DEV, dtype=torch.float32)


def _randint(lo, hi, k, g):
    return torch.randint(lo, hi, (k,), generator=g, device=DEV, dtype=torch.int64)


def _rmat_pairs(n, k, g):
    """k R-MAT draws on the smallest power of two >= n, those with an id >= n dropped."""
    scale = max(1, (n - 1).bit_length())
    us, vs = [], []
    for c0 in range(0, k, 1 << 25):
        c = min(1 << 25, k - c0)
        u = torch.zeros(c, dtype=torch.int32, device=DEV)
        v = torch.zeros(c, dtype=torch.int32, device=DEV)
        for _ in range(scale):
            r = _rand(c, g)
            sb = r >= A + B
            u.mul_(2).add_(sb)
            v.mul_(2).add_(((r >= A) & ~sb) | (r >= A + B + C))
        keep = (u < n) & (v < n)
        us.append(u[keep].to(torch.int64))
        vs.append(v[keep].to(torch.int64))
    return torch.cat(us), torch.cat(vs)


def _ws_pairs(n, k, g):
    """Ring of n vertices, every vertex joined to its k/n nearest on each side (rounded up), one
    edge in ten rewired."""
    deg = -(-k // n)
    u = torch.arange(n, device=DEV, dtype=torch.int64).repeat_interleave(deg)
    v = (u + torch.arange(1, deg + 1, device=DEV, dtype=torch.int64).repeat(n)) % n
    return u, torch.where(_rand(u.numel(), g) < 0.1, _randint(0, n, u.numel(), g), v)


def _ba_pairs(n, k, g):
    """Preferential attachment by edge copying: vertex x joins k/n earlier endpoints."""
    deg = -(-k // n)
    u = torch.arange(n, device=DEV, dtype=torch.int64).repeat_interleave(deg)
    e = torch.arange(u.numel(), device=DEV, dtype=torch.int64)
    first = (e // deg) * deg
    pos = (torch.rand(e.numel(), generator=g, device=DEV, dtype=torch.float64) *
           (2 * first).to(torch.float64)).to(torch.int64)
    ref = pos // 2
    t = torch.where((pos & 1) == 0, u[ref], -1 - ref)
    t = torch.where(first == 0, _randint(0, min(n, deg + 1), e.numel(), g), t)
    for _ in range(64):
        neg = t < 0
        if not bool(neg.any()):
            break
        t = torch.where(neg, t[(-1 - t).clamp(min=0)], t)
    return u, t


def _er_pairs(n, k, g):
    return _randint(0, n, k, g), _randint(0, n, k, g)


_FAMILY = {"rmat": _rmat_pairs, "ws": _ws_pairs, "ba": _ba_pairs, "er": _er_pairs}


def _edges(case, seed):
    """int32 [m, 2]: exactly m distinct undirected edges, shuffled, randomly oriented; twice as
    many rows when the case lists both directions."""
    n, m = case["n"], case["m"]
    g = _gen(seed)
    pairs = _FAMILY[case["family"]]
    relabel = torch.randperm(n, generator=g, device=DEV) if case["family"] == "rmat" else None
    keys, want = None, m
    while keys is None or keys.numel() < m:
        if keys is not None and case["family"] in ("ws", "ba"):
            pairs = _er_pairs  # what deduplication took is made up by random pairs
        u, v = pairs(n, int(want * 1.15) + 64 if pairs in (_rmat_pairs, _er_pairs) else want, g)
        if relabel is not None and pairs is _rmat_pairs:
            u, v = relabel[u], relabel[v]
        key = torch.minimum(u, v) * n + torch.maximum(u, v)
        key = key[u != v]
        del u, v
        keys = torch.unique(key if keys is None else torch.cat([keys, key]))
        del key
        want = max(m - keys.numel(), m // 16)
    keys = keys[torch.randperm(keys.numel(), generator=g, device=DEV)[:m]]
    u = torch.div(keys, n, rounding_mode="floor").to(torch.int32)
    v = (keys - u.to(torch.int64) * n).to(torch.int32)
    del keys
    swap = _rand(m, g) < 0.5
    e = torch.stack([torch.where(swap, v, u), torch.where(swap, u, v)], dim=1)
    del u, v, swap
    if case["both"]:
        e = torch.cat([e, e.flip(1)])[torch.randperm(2 * m, generator=g, device=DEV)]
    return e.contiguous()


def _batch_sizes(case):
    """Per graph: vertices (log-uniform), neighbours added per vertex, and the family; the same
    for every seed, so that only the edges differ."""
    k = case["graphs"]
    g = _gen(k)
    r = torch.rand(3, k, generator=g, device=DEV, dtype=torch.float64)
    lo, hi = math.log(case["n_min"]), math.log(case["n_max"])
    n = torch.exp(lo + r[0] * (hi - lo)).round().to(torch.int64)
    d = case["deg_min"] + r[1] * (case["deg_max"] - case["deg_min"])
    return n, (d / 2).round().to(torch.int64).clamp(min=1), r[2] < 0.5


def _csr(u, v, off, N):
    """The batched format from distinct undirected pairs of union ids (off: vertex offsets)."""
    G = off.numel() - 1
    key = torch.sort(torch.cat([u * N + v, v * N + u])).values
    src = torch.div(key, N, rounding_mode="floor")
    grow = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    grow[1:] = torch.cumsum(torch.bincount(src, minlength=N), 0)
    adj_off = grow[off]
    g_of = torch.repeat_interleave(torch.arange(G, device=DEV), off[1:] - off[:-1])
    col = (key - src * N - off[g_of[src]]).to(torch.int32)
    gidx = torch.repeat_interleave(torch.arange(G, device=DEV), off[1:] - off[:-1] + 1)
    pos = torch.arange(N + G, device=DEV) - gidx
    row_ptr = (grow[pos] - adj_off[gidx]).to(torch.int32)
    return api.Batch(off, adj_off, row_ptr, col, G, N, int(key.numel()))


def _batch(case, seed):
    """Half preferential-attachment, half small-world graphs, built together as one union."""
    g = _gen(seed)
    n, k, is_ba = _batch_sizes(case)
    k = torch.minimum(k, torch.div(n - 1, 2, rounding_mode="floor").clamp(min=1))
    off = torch.zeros(case["graphs"] + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(n, 0)
    N = int(off[-1])
    gv = torch.repeat_interleave(torch.arange(case["graphs"], device=DEV), n)
    kv = k[gv]
    u = torch.repeat_interleave(torch.arange(N, device=DEV), kv)  # union id of the first end
    start = torch.cumsum(kv, 0) - kv                              # first edge of every vertex
    ge = gv[u]
    j = torch.arange(u.numel(), device=DEV) - start[u]
    base, ne = off[ge], n[ge]
    local = u - base
    far = base + (torch.rand(u.numel(), generator=g, device=DEV, dtype=torch.float64) *
                  ne.to(torch.float64)).to(torch.int64).clamp(max=1 << 40)
    ring = torch.where(_rand(u.numel(), g) < 0.1, far, base + (local + j + 1) % ne)
    del far
    # preferential attachment: an endpoint of an earlier edge of the same graph
    ebase = start[off[:-1]][ge]
    prev = start[u] - ebase
    pos = (torch.rand(u.numel(), generator=g, device=DEV, dtype=torch.float64) *
           (2 * prev).to(torch.float64)).to(torch.int64)
    ref = ebase + torch.div(pos, 2, rounding_mode="floor")
    copy = torch.where((pos & 1) == 0, u[ref], -1 - ref)
    copy = torch.where(prev == 0, base + torch.minimum(j + 1, ne - 1), copy)
    del pos, ref, prev, ebase, j, local, ne, base
    ba = is_ba[ge]
    v = torch.where(ba, copy, ring)
    del copy, ring, ba, ge
    for _ in range(64):
        neg = v < 0
        if not bool(neg.any()):
            break
        v = torch.where(neg, v[(-1 - v).clamp(min=0)], v)
    key = (torch.minimum(u, v) * N + torch.maximum(u, v))[u != v]
    del u, v
    key = torch.unique(key)
    a = torch.div(key, N, rounding_mode="floor")
    return _csr(a, key - a * N, off, N)


def _serve_scales(case):
    lo, hi, k = case["scale_min"], case["scale_max"], case["graphs"]
    return [lo + (i * (hi - lo + 1)) // k if k > 1 else hi for i in range(k)]


def _serve_requests(case, seed):
    """Edge arrays of the waiting requests: R-MAT graphs, scales spread over the range."""
    return [(_edges({"family": "rmat", "n": 1 << s, "m": int(case["ef"] * (1 << s)),
                     "both": False}, seed * 1009 + i), 1 << s)
            for i, s in enumerate(_serve_scales(case))]


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "batch":
        b = _batch(case, seed)
        state["batch"] = b
        if case["plan"]:
            state["plan"] = api.BatchPlan(b.G, b.n_total, b.adj_total,
                                          {"chunk_e": 512, "items_k": 64, "light_max": 64},
                                          device=DEV)
        return state
    if kind == "serve":
        reqs = _serve_requests(case, seed)
        vo, eo = [0], [0]
        for e, n in reqs:
            vo.append(vo[-1] + n)
            eo.append(eo[-1] + e.shape[0])
        state["edges"] = torch.cat([e for e, _ in reqs])
        state["vtx_off"] = torch.tensor(vo, dtype=torch.int64, device=DEV)
        state["edge_off"] = torch.tensor(eo, dtype=torch.int64, device=DEV)
        state["n_total"] = vo[-1]
        return state
    state["edges"] = _edges(case, seed)
    if kind == "step":  # the workspace that a program counting graph after graph keeps
        state["workspace"] = api.alloc_workspace(case["n"], case["m"], device=DEV)
    elif kind == "resident":
        state["prepared"] = api.Prepared(state["edges"], case["n"])
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "count":
        if case["blocking"]:
            return api.count(state["edges"], case["n"], case["both"])
        r = api.count_async(state["edges"], case["n"], case["both"])
        return {"total": r.total, "status": r.status}
    if kind == "per_vertex":
        r = api.count_async(state["edges"], case["n"], case["both"], per_vertex=True)
        return {"total": r.total, "status": r.status, "per_vertex": r.per_vertex}
    if kind == "step":
        p = api.Prepared(state["edges"], case["n"], workspace=state["workspace"])
        r = p.count_async()
        return {"total": r.total, "status": r.status}
    if kind == "resident":
        r = state["prepared"].count_async()
        return {"total": r.total, "status": r.status}
    if kind == "batch":
        if case["plan"]:
            r = state["plan"].run_async(state["batch"], per_vertex=case["per_vertex"])
        else:
            r = api.count_batched_async(state["batch"], per_vertex=case["per_vertex"])
        out = {"totals": r.totals, "status": r.status}
        if case["per_vertex"]:
            out["per_vertex"] = r.per_vertex
        return out
    packed = api.pack_edges_async(state["edges"], state["vtx_off"], state["edge_off"],
                                  state["n_total"])
    r = api.count_batched_async(packed.batch)
    return {"totals": r.totals, "status": r.status, "pack_status": packed.status,
            "adj_off": packed.batch.adj_off, "row_ptr": packed.batch.row_ptr,
            "col": packed.batch.col}


# ------------------------------------------------------------------ bounds


def work(case):
    """Bytes of the input read once and the outputs written once; one intersection (an integer
    operation at the least) per edge."""
    kind = case["kind"]
    if kind == "batch":
        lo, hi = math.log(case["n_min"]), math.log(case["n_max"])
        n = (case["n_max"] - case["n_min"]) / (hi - lo) if hi > lo else case["n_min"]
        N = case["graphs"] * n
        m = N * (case["deg_min"] + case["deg_max"]) / 4
        out = 12 * case["graphs"] + (8 * N if case["per_vertex"] else 0)
        return {"bytes": int(8 * m + 4 * N + 16 * case["graphs"] + out), "flops": int(m)}
    if kind == "serve":
        m = sum(int(case["ef"] * (1 << s)) for s in _serve_scales(case))
        n = sum(1 << s for s in _serve_scales(case))
        return {"bytes": int(16 * m + 4 * n + 40 * case["graphs"]), "flops": int(m)}
    entries = case["m"] * (2 if case["both"] else 1)
    out = 12 + (8 * case["n"] if kind == "per_vertex" else 0)
    # a prepared graph is its node and neighbour arrays
    data = 4 * case["m"] + 4 * case["n"] if kind == "resident" else 8 * entries
    return {"bytes": int(data + out), "flops": int(case["m"])}


# ------------------------------------------------------------------ exact counts


def _wedge_counts(u, v, n, per_vertex):
    """(triangles, per-vertex counts or None) of distinct undirected pairs, by testing every
    wedge of the degree-ordered graph; None when there are too many wedges."""
    deg = torch.bincount(torch.cat([u, v]), minlength=n)
    swap = (deg[u] > deg[v]) | ((deg[u] == deg[v]) & (u > v))
    key = torch.sort(torch.where(swap, v, u) * n + torch.where(swap, u, v)).values
    s = torch.div(key, n, rounding_mode="floor")
    t = key - s * n
    end = torch.cumsum(torch.bincount(s, minlength=n), 0)
    left = end[s] - 1 - torch.arange(key.numel(), device=DEV)
    cum = torch.cumsum(left, 0)
    if key.numel() == 0 or int(cum[-1]) > 3_000_000_000:
        return None
    total = 0
    pv = torch.zeros(n, dtype=torch.int64, device=DEV) if per_vertex else None
    step, lo, wedges = 1 << 26, 0, int(cum[-1])
    while lo < wedges:
        hi = min(lo + step, wedges)
        w = torch.arange(lo, hi, device=DEV)
        i = torch.searchsorted(cum, w, right=True)
        j = i + 1 + (w - (cum[i] - left[i]))
        a, b = t[i], t[j]
        # the closing edge in its degree order
        sw = (deg[a] > deg[b]) | ((deg[a] == deg[b]) & (a > b))
        q = torch.where(sw, b, a) * n + torch.where(sw, a, b)
        p = torch.searchsorted(key, q).clamp(max=key.numel() - 1)
        hit = key[p] == q
        total += int(hit.sum())
        if per_vertex:
            pv += torch.bincount(torch.cat([s[i][hit], a[hit], b[hit]]), minlength=n)
        lo = hi
    return total, pv


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        b = _batch(case, seed)
        N = b.n_total
        g_of = torch.repeat_interleave(torch.arange(b.G, device=DEV),
                                       b.vtx_off[1:] - b.vtx_off[:-1])
        first = torch.arange(N, device=DEV) + g_of
        lens = (b.row_ptr[first + 1] - b.row_ptr[first]).to(torch.int64)
        src = torch.repeat_interleave(torch.arange(N, device=DEV), lens)
        dst = b.col.to(torch.int64) + b.vtx_off[g_of[src]]
        keep = src < dst
        r = _wedge_counts(src[keep], dst[keep], N, True)
        if r is None:
            return None
        totals = torch.zeros(b.G, dtype=torch.int64, device=DEV).index_add_(0, g_of, r[1]) // 3
        out = {"totals": totals, "status": None}
        if case["per_vertex"]:
            out["per_vertex"] = r[1]
        return out
    if kind == "serve":
        reqs = _serve_requests(case, seed)
        totals, ends = [], [0]
        for e, n in reqs:
            r = _wedge_counts(e[:, 0].to(torch.int64), e[:, 1].to(torch.int64), n, False)
            if r is None:
                return None
            totals.append(r[0])
            ends.append(ends[-1] + 2 * e.shape[0])
        return {"totals": torch.tensor(totals, dtype=torch.int64, device=DEV), "status": None,
                "pack_status": None, "adj_off": torch.tensor(ends, dtype=torch.int64, device=DEV),
                "row_ptr": None, "col": None}
    if case["m"] > 20_000_000:
        return None
    e = _edges(dict(case, both=False), seed).to(torch.int64)
    r = _wedge_counts(e[:, 0], e[:, 1], case["n"], kind == "per_vertex")
    if r is None:
        return None
    if kind == "count" and case["blocking"]:
        return r[0]
    out = {"total": torch.tensor([r[0]], dtype=torch.int64, device=DEV), "status": None}
    if kind == "per_vertex":
        out["per_vertex"] = r[1]
    return out
