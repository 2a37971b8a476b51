"""GPU parity of the batched entry points (tc_count_batched, tc_batched_plan_*) against the
CPU oracle, graph by graph, bit-exact: per-graph totals and per-vertex counts, invalid graphs
reported per graph without disturbing the others, and a captured plan replayed several times
with other GPU work in between."""
import hashlib
import json
import os

import numpy as np
import pytest
import torch

import oracle
from paper_1503_00576_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def as_batch(packed) -> api.Batch:
    return api.Batch(packed["vtx_off"].to(DEV), packed["adj_off"].to(DEV),
                     packed["row_ptr"].to(DEV), packed["col"].to(DEV), packed["G"],
                     packed["n_total"], packed["adj_total"])


def mixed_graphs(seed=0, count=48):
    rng = np.random.default_rng(seed)
    gs = []
    for i in range(count):
        kind = i % 4
        n = int(rng.integers(2, 3000))
        if kind == 0:
            gs.append((synth.barabasi_albert(n, int(rng.integers(1, 12)), seed * 1000 + i), n))
        elif kind == 1:
            gs.append((synth.watts_strogatz(max(n, 3), int(rng.integers(1, 10)), 0.1, i), max(n, 3)))
        elif kind == 2:
            gs.append((synth.erdos_renyi(min(n, 400), float(rng.choice([0.02, 0.1, 0.5])), i), min(n, 400)))
        else:
            s = int(rng.integers(4, 11))
            gs.append(synth.rmat_graph(s, 16, seed=i))
    gs.append((torch.zeros((0, 2), dtype=torch.int32), 7))      # isolated vertices only
    gs.append((torch.zeros((0, 2), dtype=torch.int32), 1))
    k = 40
    gs.append((torch.tensor([(i, j) for i in range(k) for j in range(i + 1, k)], dtype=torch.int32), k))
    # dense graph: forward degrees up to ~600, above the edge-per-lane path's 256
    gs.append((synth.erdos_renyi(700, 0.9, seed * 7 + 1), 700))
    return gs


def oracle_per_graph(gs):
    out = []
    for e, n in gs:
        t, pv = oracle.count(e, n, per_vertex=True)
        out.append((t, pv))
    return out


def check(res: api.BatchResult, gs, want, per_vertex=True):
    tot = res.totals.cpu().numpy().astype(np.uint64)
    assert not res.status.cpu().numpy().any()
    for g, (t, _) in enumerate(want):
        assert tot[g] == t, g
    if per_vertex:
        pv = res.per_vertex.cpu().numpy().astype(np.uint64)
        assert np.array_equal(pv, np.concatenate([p for _, p in want]))


def test_batched_one_shot():
    gs = mixed_graphs(1)
    want = oracle_per_graph(gs)
    b = as_batch(synth.pack_symmetric(gs))
    check(api.count_batched(b, per_vertex=True), gs, want)
    check(api.count_batched(b, per_vertex=False), gs, want, per_vertex=False)


def test_batched_union_additive():
    gs = mixed_graphs(2, 24)
    b = as_batch(synth.pack_symmetric(gs))
    res = api.count_batched(b)
    off, parts = 0, []
    for e, n in gs:
        parts.append(e.numpy().astype(np.int64) + off)
        off += n
    assert int(res.totals.sum()) == oracle.count(np.concatenate(parts), off)


@pytest.mark.parametrize("tuning", [None, {"items_k": 16, "wgs_per_cu": 1}, {"items_k": 1024},
                                    {"chunk_e": 64, "wgs_per_cu": 1}, {"chunk_e": 1536}])
def test_plan_replays(tuning):
    """A captured plan replayed several times, with eager GPU work in between, every replay
    equal to the one-shot result; then a smaller batch through the same plan."""
    gs = mixed_graphs(3)
    want = oracle_per_graph(gs)
    b = as_batch(synth.pack_symmetric(gs))
    plan = api.BatchPlan(b.G + 5, b.n_total + 100, b.adj_total + 1000, tuning, device=DEV)
    for rep in range(4):
        res = plan.run_async(b, per_vertex=(rep % 2 == 1))
        x = torch.randn(1 << 20, device=DEV)          # unrelated eager work
        (x * 2).sum().item()
        torch.cuda.synchronize()
        check(res, gs, want, per_vertex=(rep % 2 == 1))
    small = gs[5:17]
    b2 = as_batch(synth.pack_symmetric(small))
    res2 = plan.run_async(b2, per_vertex=True)
    torch.cuda.synchronize()
    check(res2, small, oracle_per_graph(small))
    res3 = plan.run_async(b, per_vertex=False)
    torch.cuda.synchronize()
    check(res3, gs, want, per_vertex=False)
    plan.close()


def test_batched_bad_graphs_reported_per_graph():
    gs = mixed_graphs(4, 8)
    packed = synth.pack_symmetric(gs)
    col = packed["col"].clone()
    vo, ao = packed["vtx_off"], packed["adj_off"]
    rp = packed["row_ptr"]
    # graph 1: swap two entries of a row with at least two entries -> unsorted
    g = 1
    v0 = int(vo[g]); n = int(vo[g + 1] - v0)
    base = int(ao[g])
    for x in range(n):
        r0, r1 = int(rp[v0 + g + x]), int(rp[v0 + g + x + 1])
        if r1 - r0 >= 2:
            a, c = base + r0, base + r0 + 1
            col[a], col[c] = col[c].clone(), col[a].clone()
            break
    # graph 3: an id out of range
    g3 = 3
    col[int(ao[g3])] = int(vo[g3 + 1] - vo[g3]) + 5
    packed["col"] = col
    b = as_batch(packed)
    res = api.BatchPlan(b.G, b.n_total, b.adj_total, device=DEV).run_async(b)
    torch.cuda.synchronize()
    st = res.status.cpu().numpy()
    assert st[1] == api.E_UNSORTED and st[3] == api.E_RANGE
    want = oracle_per_graph(gs)
    tot = res.totals.cpu().numpy().astype(np.uint64)
    for gg in range(len(gs)):
        if gg not in (1, 3):
            assert st[gg] == 0 and tot[gg] == want[gg][0]


def test_batched_asymmetric():
    gs = [(torch.tensor([(0, 1), (1, 2), (0, 2)], dtype=torch.int32), 3)]
    packed = synth.pack_symmetric(gs)
    # drop the mirror (2 -> 0): rows 0:[1,2] 1:[0,2] 2:[1] ; rebuild by hand
    packed["row_ptr"] = torch.tensor([0, 2, 4, 5], dtype=torch.int32)
    packed["col"] = torch.tensor([1, 2, 0, 2, 1], dtype=torch.int32)
    packed["adj_off"] = torch.tensor([0, 5], dtype=torch.int64)
    packed["adj_total"] = 5
    b = as_batch(packed)
    with pytest.raises(api.TCError) as ei:
        api.count_batched(b)
    assert ei.value.name == "asymmetric"


def asymmetric_even_rows(seed):
    """Sorted rows on 6 vertices that are not symmetric although the entries number exactly
    twice the forward entries (so only the symmetry sum can tell)."""
    rng = np.random.default_rng(seed)
    while True:
        rows = [sorted(set(rng.choice([y for y in range(6) if y != x], size=int(rng.integers(0, 4)),
                                      replace=False).tolist())) for x in range(6)]
        deg = [len(r) for r in rows]
        fwd = sum(1 for x in range(6) for y in rows[x] if (deg[y], y) > (deg[x], x))
        ents = {(x, y) for x in range(6) for y in rows[x]}
        if 2 * fwd == len(ents) and any((y, x) not in ents for x, y in ents):
            return rows


def test_batched_asymmetric_even_count():
    gs = mixed_graphs(5, 4)
    packed = synth.pack_symmetric(gs)
    G = packed["G"]
    rows = asymmetric_even_rows(11)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    col = np.array([y for r in rows for y in r], dtype=np.int32)
    # append the bad graph as graph G
    packed["vtx_off"] = torch.cat([packed["vtx_off"], packed["vtx_off"][-1:] + 6])
    packed["adj_off"] = torch.cat([packed["adj_off"], packed["adj_off"][-1:] + len(col)])
    packed["row_ptr"] = torch.cat([packed["row_ptr"], torch.from_numpy(rp)])
    packed["col"] = torch.cat([packed["col"], torch.from_numpy(col)])
    packed["G"] = G + 1
    packed["n_total"] += 6
    packed["adj_total"] += len(col)
    b = as_batch(packed)
    res = api.BatchPlan(b.G, b.n_total, b.adj_total, device=DEV).run_async(b)
    torch.cuda.synchronize()
    st = res.status.cpu().numpy()
    assert st[G] == api.E_ASYMMETRIC and not st[:G].any()
    want = oracle_per_graph(gs)
    tot = res.totals.cpu().numpy().astype(np.uint64)
    assert all(tot[g] == want[g][0] for g in range(G))


def test_batch_spec_sample():
    """A slice of the 4096-graph benchmark batch (Barabasi-Albert / Watts-Strogatz mix)."""
    spec = synth.BatchSpec(graphs=32, seed=7)
    gs = synth.batch_graphs(spec)
    want = oracle_per_graph(gs)
    b = as_batch(synth.pack_symmetric(gs, device=DEV))
    check(api.count_batched(b, per_vertex=True), gs, want)


# every form of the batched counting kernel, forced on small graphs through the plan tuning:
# all rows heavy (bitmap, sorted LDS list, sorted list in global memory), a low light/heavy
# threshold with mixed forms, and heavy items of 16 out-neighbours
FORCED = {
    "heavy_bitmap": {"light_max": 0},
    "heavy_lds_list": {"light_max": 0, "bitmap_span": 0},
    "heavy_global_list": {"light_max": 0, "bitmap_span": 0, "list_max": 0},
    "mixed": {"light_max": 8, "bitmap_span": 50, "list_max": 20},
    "small_items": {"light_max": 4, "items_k": 16, "bitmap_span": 200, "list_max": 12},
}


@pytest.mark.parametrize("name", sorted(FORCED))
def test_batched_forced_forms(name):
    gs = mixed_graphs(6, 24)
    want = oracle_per_graph(gs)
    b = as_batch(synth.pack_symmetric(gs))
    plan = api.BatchPlan(b.G, b.n_total, b.adj_total, FORCED[name], device=DEV)
    for pv in (True, False):
        res = plan.run_async(b, per_vertex=pv)
        torch.cuda.synchronize()
        check(res, gs, want, per_vertex=pv)
    plan.close()


# ------------------------------------------------------------------ edge arrays -> batch


def pack_on_device(gs):
    """tc_batched_pack of graphs [(edges int32 [m, 2], n), ...] (edges may hold bad ids)."""
    ns = [n for _, n in gs]
    ms = [int(e.shape[0]) for e, _ in gs]
    vo = torch.tensor(np.concatenate([[0], np.cumsum(ns)]), dtype=torch.int64, device=DEV)
    eo = torch.tensor(np.concatenate([[0], np.cumsum(ms)]), dtype=torch.int64, device=DEV)
    edges = torch.cat([e.to(torch.int32) for e, _ in gs]).reshape(-1, 2).to(DEV)
    return api.pack_edges_async(edges, vo, eo, int(sum(ns)))


def test_pack_matches_symmetric_csr():
    """The device pack gives exactly the symmetric CSR (rows ascending, local ids) that the
    input generator's host-side formatter builds, including empty graphs and graphs without
    edges."""
    gs = mixed_graphs(7, 20)
    gs.insert(3, (torch.zeros((0, 2), dtype=torch.int32), 0))   # a graph without vertices
    gs.append((torch.zeros((0, 2), dtype=torch.int32), 0))
    p = pack_on_device(gs)
    torch.cuda.synchronize()
    assert not p.status.cpu().numpy().any()
    want = synth.pack_symmetric(gs)
    A = int(want["adj_total"])
    assert torch.equal(p.batch.adj_off.cpu(), want["adj_off"])
    assert torch.equal(p.batch.row_ptr.cpu(), want["row_ptr"])
    assert torch.equal(p.batch.col.cpu()[:A], want["col"])
    res = api.count_batched(p.batch, per_vertex=True)
    check(res, gs, oracle_per_graph(gs))


@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_pack_bad_ids_reported_per_graph(where):
    """An id outside [0, n_g) or a self-loop fails only its own graph (pack status), whatever
    its position; the other graphs' counts are exact."""
    gs = mixed_graphs(8, 10)
    bad = {"first": 0, "middle": 5, "last": len(gs) - 1}[where]
    e, n = gs[bad]
    gs[bad] = (torch.cat([e, torch.tensor([[0, n + 3]], dtype=torch.int32)]), n)
    gs[(bad + 2) % len(gs)] = (torch.tensor([[1, 1], [0, 1]], dtype=torch.int32), 3)
    p = pack_on_device(gs)
    res = api.count_batched_async(p.batch)
    torch.cuda.synchronize()
    pst = p.status.cpu().numpy()
    assert pst[bad] == api.E_RANGE
    assert pst[(bad + 2) % len(gs)] == api.E_SELF_LOOP
    st = res.status.cpu().numpy()
    tot = res.totals.cpu().numpy().astype(np.uint64)
    for g, (e, n) in enumerate(gs):
        if g in (bad, (bad + 2) % len(gs)):
            continue
        assert pst[g] == 0 and st[g] == 0
        assert tot[g] == oracle.count(e, n)


def test_pack_offsets_not_prefix_sums():
    """Offsets that are not prefix sums mark every graph of the batch; nothing else breaks."""
    gs = mixed_graphs(9, 4)
    ns = [n for _, n in gs]
    ms = [int(e.shape[0]) for e, _ in gs]
    vo = np.concatenate([[0], np.cumsum(ns)]).astype(np.int64)
    vo[2] = vo[3] + 5  # decreasing
    eo = np.concatenate([[0], np.cumsum(ms)]).astype(np.int64)
    edges = torch.cat([e for e, _ in gs]).to(DEV)
    p = api.pack_edges_async(edges, torch.from_numpy(vo).to(DEV), torch.from_numpy(eo).to(DEV),
                             int(sum(ns)))
    torch.cuda.synchronize()
    assert (p.status.cpu().numpy() == api.E_ARG).all()


def test_batch4096_golden():
    """The benchmark's full batch (4096 Barabasi-Albert / Watts-Strogatz graphs, 13.7M
    vertices, 122M edges) through a tuned-size plan: every graph's total and the whole
    per-vertex array (digest) against the oracle's stored values."""
    with open(os.path.join(os.path.dirname(__file__), "golden", "batch4096.json")) as f:
        ref = json.load(f)
    graphs = synth.batch_graphs(synth.BatchSpec(graphs=4096, seed=0), device=DEV)
    h = hashlib.sha256()
    for e, n in graphs:
        h.update(np.int64(n).tobytes())
        h.update(np.ascontiguousarray(e.cpu().numpy()).tobytes())
    assert h.hexdigest() == ref["inputs_sha256"]
    b = as_batch(synth.pack_symmetric(graphs, device=DEV))
    del graphs
    plan = api.BatchPlan(b.G, b.n_total, b.adj_total, {"chunk_e": 512}, device=DEV)
    res = plan.run_async(b, per_vertex=True)
    torch.cuda.synchronize()
    res.check()
    assert res.totals.cpu().tolist() == ref["totals"]
    pv = res.per_vertex.cpu().numpy()
    assert int(pv.sum()) == ref["per_vertex_sum"]
    assert hashlib.sha256(pv.astype("<u8").tobytes()).hexdigest() == ref["per_vertex_sha256"]
    res2 = plan.run_async(b)
    torch.cuda.synchronize()
    assert res2.totals.cpu().tolist() == ref["totals"]
    plan.close()


def test_autotune_batched(tmp_path):
    """The batched tuner (chunk size, heavy item size, light/heavy threshold) returns one of
    its candidates, which counts exactly, and caches it by device, sizes and degree profile."""
    from paper_1503_00576_amd import autotune
    gs = mixed_graphs(10, 16)
    want = oracle_per_graph(gs)
    b = as_batch(synth.pack_symmetric(gs))
    cands = [{"chunk_e": 256, "items_k": 64, "light_max": 64},
             {"chunk_e": 1024, "items_k": 256, "light_max": 256}]
    cache = str(tmp_path / "tune.json")
    best, timings = autotune.tune_batched(b, reps=1, cache=cache, candidates=cands)
    assert best in cands and len(timings) == 2
    plan = api.BatchPlan(b.G, b.n_total, b.adj_total, best, device=DEV)
    res = plan.run_async(b, per_vertex=True)
    torch.cuda.synchronize()
    check(res, gs, want)
    plan.close()
    assert autotune.tune_batched(b, cache=cache, candidates=cands[:1])[0] == best


@pytest.mark.parametrize("where", [1, 62, 63, 64, 65, 127, 128, 255, 256])
def test_bad_order_at_walk_steps(where):
    """A descending and a repeated pair at the setup walk's step and lane edges, in the middle
    graph of three: reported for that graph only."""
    k = 300
    star = torch.tensor([(0, x) for x in range(1, k)], dtype=torch.int32)
    gs = [synth.watts_strogatz(20, 3, 0.1, 5), star, synth.watts_strogatz(33, 4, 0.1, 6)]
    gs = [(gs[0], 20), (gs[1], k), (gs[2], 33)]
    want = [oracle.count(e, n) for e, n in gs]
    packed = synth.pack_symmetric(gs)
    base = int(packed["adj_off"][1])
    for kind, status in (("swap", api.E_UNSORTED), ("repeat", api.E_DUP_EDGE)):
        b = as_batch(packed)
        col = packed["col"].clone()
        if kind == "swap":
            col[base + where], col[base + where - 1] = (int(packed["col"][base + where - 1]),
                                                        int(packed["col"][base + where]))
        else:
            col[base + where] = col[base + where - 1]
        b.col = col.to(DEV)
        res = api.count_batched_async(b, per_vertex=True)
        assert res.status.tolist() == [0, status, 0]
        tot = res.totals.tolist()
        assert tot[0] == want[0] and tot[2] == want[2]


@pytest.mark.parametrize("tuning", [{"light_max": 64, "chunk_e": 64}, {"light_max": 256},
                                    {"light_max": 255, "chunk_e": 64}, {"light_max": 0},
                                    {"light_max": 2, "chunk_e": 1536, "items_k": 16}])
@pytest.mark.parametrize("many", [False, True])
def test_light_rows_at_window_edges(tuning, many):
    """Rows around light_max, windows that hold one row, waves that straddle graphs, pieces of
    1, 7, 8, 9, 16, 17 entries; few vertices per wave (small capacity) and 64 (large)."""
    gs = []
    for k in (2, 3, 8, 9, 10, 17, 18, 64, 65, 66, 256, 257, 258):
        gs.append((torch.tensor([(i, j) for i in range(k) for j in range(i + 1, k)],
                                dtype=torch.int32), k))
        gs.append((torch.zeros((0, 2), dtype=torch.int32), 1))
    gs.append((synth.erdos_renyi(300, 0.5, 3), 300))
    want = oracle_per_graph(gs)
    b = as_batch(synth.pack_symmetric(gs))
    cap = (64 * 8192 if many else b.n_total) + 1
    plan = api.BatchPlan(b.G, cap, b.adj_total, tuning, device=DEV)
    for pv in (True, False):
        check(plan.run_async(b, per_vertex=pv), gs, want, per_vertex=pv)
    plan.close()


def ring(n):
    return torch.tensor([(i, (i + 1) % n) for i in range(n)] + [(i, (i + 2) % n) for i in range(n)],
                        dtype=torch.int32), n


def splice(packed, g, row_ptr, col):
    """The batch with graph g's row offsets (its n + 1) and entries replaced."""
    vo, ao = packed["vtx_off"].tolist(), packed["adj_off"].tolist()
    n, G = len(row_ptr) - 1, packed["G"]
    grow_n, grow_a = n - (vo[g + 1] - vo[g]), len(col) - (ao[g + 1] - ao[g])
    rp = packed["row_ptr"]
    return {"G": G, "n_total": packed["n_total"] + grow_n, "adj_total": packed["adj_total"] + grow_a,
            "vtx_off": torch.tensor([v + (grow_n if k > g else 0) for k, v in enumerate(vo)]),
            "adj_off": torch.tensor([v + (grow_a if k > g else 0) for k, v in enumerate(ao)]),
            "row_ptr": torch.cat([rp[:vo[g] + g], torch.as_tensor(row_ptr, dtype=torch.int32),
                                  rp[vo[g + 1] + g + 1:]]),
            "col": torch.cat([packed["col"][:ao[g]], torch.as_tensor(col, dtype=torch.int32),
                              packed["col"][ao[g + 1]:]])}


def check_isolated(packed, want, bad):
    """Statuses E_ARG for the graphs `bad` and 0 for the others, whose counts are `want`'s: one-shot
    and in a plan with room, totals and per-vertex."""
    b = as_batch(packed)
    plan = api.BatchPlan(b.G + 3, b.n_total + 5000, 2 * b.adj_total + 100000, device=DEV)
    vo = packed["vtx_off"].tolist()
    for pv in (True, False):
        for res in (api.count_batched_async(b, per_vertex=pv), plan.run_async(b, per_vertex=pv)):
            assert res.status.tolist() == [api.E_ARG if g in bad else 0 for g in range(b.G)]
            for g, (t, per) in enumerate(want):
                if g in bad:
                    continue
                assert int(res.totals[g]) == t, g
                if pv:
                    got = res.per_vertex[vo[g]:vo[g + 1]].cpu().numpy().astype(np.uint64)
                    assert np.array_equal(got, per), g
    plan.close()


@pytest.mark.parametrize("before,after", [(5, 7), (40, 300), (3000, 2000)])
@pytest.mark.parametrize("row_ptr", [[0, 5, 3, 8], [0, 8, 0, 8], [8, 0, 8, 0], [3, 2, 1, 8]])
def test_descending_row_offsets_stay_in_their_graph(row_ptr, before, after):
    """A descent in one graph's row offsets makes its rows' lengths add up to more than its
    entries: the graph is reported, the valid ones before and after it keep status and counts."""
    gs = [ring(before), (torch.tensor([(0, 1)], dtype=torch.int32), 3), ring(after)]
    packed = splice(synth.pack_symmetric(gs), 1, row_ptr, [1, 2, 0, 2, 0, 1, 1, 2])
    check_isolated(packed, oracle_per_graph(gs), {1})


@pytest.mark.parametrize("kind", ["no forward entry", "all forward"])
def test_row_lengths_beyond_32_bits_stay_in_their_graph(kind):
    """Row offsets that swing between 0 and 65,536 over 131,071 vertices: the lengths of the rows
    that ascend add up to 2^32 - 6, six entries (the first graph's) short of a wrap.  Entries that
    name only the rows that descend, or the first vertices in order (long forward rows)."""
    k = 1 << 16
    tri = torch.tensor([(0, 1), (1, 2), (0, 2)], dtype=torch.int32)
    gs = [(tri, 3), ring(9), (tri, 3), ring(50)]
    row_ptr = np.tile(np.array([0, k], np.int32), k)
    row_ptr[0] = 6
    col = np.minimum(np.arange(k) * 2 + 1, 2 * k - 3) if kind == "no forward entry" else np.arange(k)
    packed = splice(synth.pack_symmetric(gs), 1, row_ptr, col.astype(np.int32))
    check_isolated(packed, oracle_per_graph(gs), {1})


@pytest.mark.parametrize("where,bad", [("inside the graph before", {1, 2}), ("far out", {1, 2}),
                                       ("at the start", {1, 2}), ("negative", {1, 2})])
def test_descending_adjacency_offsets_stay_in_their_graphs(where, bad):
    """One adjacency offset moved before the range of the graph that ends there: that graph
    descends, and the next one's range meets the first graph's.  Or moved out of the batch.  The
    graphs around them keep status and counts."""
    gs = [ring(40), ring(30), ring(20), ring(300), ring(5)]
    packed = dict(synth.pack_symmetric(gs))
    ao = packed["adj_off"].clone()
    ao[2] = {"inside the graph before": int(ao[1]) - 4, "far out": 1 << 40, "at the start": 0,
             "negative": -8}[where]
    packed["adj_off"] = ao
    check_isolated(packed, oracle_per_graph(gs), bad)
