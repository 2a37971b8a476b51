"""Preprocessing of small graphs (counting sorts, at most 16384 vertices and 2^18 entries) against
the general path, which sort_onesweep = 1 selects on the same graphs, and the oracle: equal
arrays and counts on both sides of the limits, and the same errors."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_00576_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GENERAL = {"sort_onesweep": 1}


def random_graph(n, m, seed):
    """m distinct edges, a crowded low end (hubs, long panels), shuffled and turned."""
    rng = np.random.default_rng(seed)
    key = np.zeros(0, np.int64)
    while len(key) < m:
        a = (n * rng.random(2 * m) ** 2).astype(np.int64)
        b = rng.integers(0, n, 2 * m)
        k = np.minimum(a, b) * n + np.maximum(a, b)
        key = np.unique(np.concatenate([key, k[a != b]]))
    key = rng.permutation(key)[:m]
    e = np.stack([key // n, key % n], 1).astype(np.int32)
    flip = rng.random(m) < 0.5
    e[flip] = e[flip][:, ::-1]
    return e


@pytest.mark.parametrize("n,m", [(2, 1), (3, 3), (63, 900), (64, 1000), (65, 1000), (255, 4095),
                                 (1000, 4096), (1000, 4097), (4096, 20000), (16383, 100000),
                                 (16384, 1 << 18), (16384, (1 << 18) + 1), (16385, 100000)])
@pytest.mark.parametrize("both", [False, True])
def test_small_path_equals_general(n, m, both):
    if both:
        m = (m + 1) // 2
    e = random_graph(n, m, n + m)
    want, pv = oracle.count(e, n, per_vertex=True)
    if both:
        e = np.concatenate([e, e[:, ::-1]])[np.random.default_rng(1).permutation(2 * m)]
    t = torch.tensor(np.ascontiguousarray(e), device=DEV)
    a = api.Prepared(t, n, both)
    b = api.Prepared(t, n, both, options=GENERAL)
    x, y = a.arrays(), b.arrays()
    for k in ("deg", "perm", "rank", "row_ptr", "col", "src"):
        assert torch.equal(x[k], y[k]), k
    for p in (a, b):
        assert p.count() == want
        r = p.count_async(per_vertex=True).check()
        assert int(r.total.item()) == want
        assert np.array_equal(r.per_vertex.cpu().numpy().astype(np.uint64), pv)
    assert api.count(t, n, both) == want


@pytest.mark.parametrize("options", [None, GENERAL, {"panel_ranks": 64}])
def test_small_graph_errors(options):
    base = synth.watts_strogatz(200, 5, 0.1, 3).numpy()
    cases = [([[5, 5]], "self_loop"), ([[0, 200]], "range"), ([[-1, 3]], "range"),
             (base[:1], "dup_edge"), (base[7:8, ::-1], "dup_edge")]
    for extra, name in cases:
        e = torch.tensor(np.concatenate([base, np.array(extra, np.int32)]), device=DEV)
        with pytest.raises(api.TCError) as ei:
            api.count(e, 200, options=options)
        assert ei.value.name == name
    both = np.concatenate([base, base[:, ::-1]])
    swapped = both.copy()
    swapped[0] = swapped[0][::-1]  # an edge twice in one direction
    with pytest.raises(api.TCError) as ei:
        api.count(torch.tensor(swapped, device=DEV), 200, both=True, options=options)
    assert ei.value.name in ("asymmetric", "dup_edge")
    assert api.count(torch.tensor(both, device=DEV), 200, both=True, options=options) == \
        oracle.count(base, 200)


def test_many_repeats_of_one_edge():
    """A row far longer than a simple graph's (reported, not sorted)."""
    e = torch.tensor([[0, 1]] * 5000 + [[1, 2], [0, 2]], dtype=torch.int32, device=DEV)
    for options in (None, GENERAL):
        with pytest.raises(api.TCError) as ei:
            api.count(e, 3, options=options)
        assert ei.value.name == "dup_edge"


def test_small_path_in_a_captured_graph():
    """A count recorded into a HIP graph and replayed, with other work in between."""
    e = torch.tensor(random_graph(3000, 20000, 5), device=DEV)
    want = oracle.count(e.cpu().numpy(), 3000)
    ws = api.alloc_workspace(3000, 20000, device=DEV)
    out = api.Result(torch.zeros(1, dtype=torch.int64, device=DEV),
                     torch.zeros(1, dtype=torch.int32, device=DEV))
    api.count_async(e, 3000, workspace=ws, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        api.count_async(e, 3000, workspace=ws, out=out)
    for _ in range(4):
        out.total.fill_(-1)
        g.replay()
        assert int(out.total.item()) == want and int(out.status.item()) == 0
        torch.randn(1 << 16, device=DEV).sum().item()


def guarded(n):
    """int64[n] between two guards of 4096 words of -7"""
    room = torch.full((n + 8192,), -7, dtype=torch.int64, device=DEV)
    return room, room[4096:4096 + n]


@pytest.mark.parametrize("n", [200, 16384, 20000])
@pytest.mark.parametrize("kind", ["range", "self_loop", "dup_edge", "asymmetric"])
def test_per_vertex_counts_after_an_error(kind, n):
    """The order of the vertices is missing after an error: the counts are zeros and nothing beside
    them is written, whatever the workspace held before."""
    base = synth.watts_strogatz(200, 5, 0.1, 3).numpy()
    extra = {"range": [[0, n]], "self_loop": [[5, 5]], "dup_edge": base[:1, ::-1],
             "asymmetric": base[:2]}[kind]
    both = kind == "asymmetric"
    e = torch.tensor(np.concatenate([base, np.array(extra, np.int32)]), device=DEV)
    if both and e.shape[0] % 2:
        e = e[1:].contiguous()
    ws = api.alloc_workspace(n, e.shape[0], both, DEV).fill_(0xFF)
    room, pv = guarded(n)
    out = api.Result(torch.empty(1, dtype=torch.int64, device=DEV),
                     torch.empty(1, dtype=torch.int32, device=DEV), pv)
    api.count_async(e, n, both, per_vertex=True, workspace=ws, out=out)
    assert api.STATUS_NAMES[int(out.status.item())] == kind
    assert not pv.any()
    assert (room[:4096] == -7).all() and (room[4096 + n:] == -7).all()


def test_per_vertex_counts_on_a_mismatched_workspace():
    """Prepared for 200 vertices, counted as a graph of 3000."""
    e = synth.watts_strogatz(200, 5, 0.1, 3).to(DEV)
    ws = api.alloc_workspace(3000, 9000, device=DEV).fill_(0xFF)
    p = api.Prepared(e, 200, workspace=ws)
    p.n, p.m = 3000, 9000
    room, pv = guarded(3000)
    out = api.Result(torch.empty(1, dtype=torch.int64, device=DEV),
                     torch.empty(1, dtype=torch.int32, device=DEV), pv)
    p.count_async(per_vertex=True, out=out)
    assert int(out.status.item()) == api.E_MISMATCH
    assert not pv.any()
    assert (room[:4096] == -7).all() and (room[4096 + 3000:] == -7).all()


@pytest.mark.parametrize("n,m", [(16000, 250000), (40000, 900000), (1 << 18, 2000000)])
@pytest.mark.parametrize("every", [1, 997])
def test_repeated_edges_in_many_rows(n, m, every):
    """Repeated edges all over the rows, found by many workgroups of the row sorts while others of
    the same launch begin, rows beyond one wave's among them: reported each time, and the same
    workspace then counts a valid graph."""
    e = random_graph(n, m, m + n)
    hub = n - 1 - (np.arange(2200, dtype=np.int32))
    clique = np.stack(np.triu_indices(1100, 1), 1).astype(np.int32) if n > 16384 else e[:0]
    good = np.unique(np.sort(np.concatenate([e, np.stack([hub[1:], hub[:-1]], 1), clique]), 1), axis=0)
    want = oracle.count(good, n)
    bad = np.concatenate([good, good[::every, ::-1]])
    bad = torch.tensor(bad[np.random.default_rng(every).permutation(len(bad))], device=DEV)
    good = torch.tensor(good, device=DEV)
    ws = api.alloc_workspace(n, bad.shape[0], device=DEV)
    for _ in range(10):
        out = api.count_async(bad, n, workspace=ws)
        assert int(out.status.item()) == api.E_DUP_EDGE
    assert int(api.count_async(good, n, workspace=ws).check().total.item()) == want
