"""The scans and radix passes at the edges of their tiles and of the rules that choose their
launches (GPU, exact): the sort against torch's stable sort, whole counts against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_00576_amd import api

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TILE, RAW = 8192, 128  # keys per tile; up to RAW tiles a pass reads the unscanned table


@pytest.mark.parametrize("count", [1, 2, TILE - 1, TILE, TILE + 1, 64 * TILE, 64 * TILE + 1,
                                   65 * TILE, RAW * TILE, RAW * TILE + 1, 3 * RAW * TILE - 5])
@pytest.mark.parametrize("bits", [8, 21])
def test_sort_at_tile_edges(count, bits):
    gen = torch.Generator().manual_seed(count + bits)
    keys = torch.randint(0, 1 << 40, (count,), generator=gen, dtype=torch.int64)
    keys[: count // 3] &= ~0xFF  # a crowded digit
    want = keys[torch.argsort(keys & ((1 << bits) - 1), stable=True)]
    got = api.sort_u64(keys.to(DEV), bits).cpu()
    assert torch.equal(got, want)


@pytest.mark.parametrize("bits", [9, 17, 18, 19, 25, 27, 28])
@pytest.mark.parametrize("count", [TILE + 1, RAW * TILE, RAW * TILE + 1])
def test_sort_with_wide_digits(bits, count):
    """Widths on both sides of the ones that take digits of 9 bits."""
    gen = torch.Generator().manual_seed(count + bits)
    keys = torch.randint(0, 1 << 40, (count,), generator=gen, dtype=torch.int64)
    keys[: count // 3] &= ~0x1FF  # a crowded digit
    keys[count // 2:] |= 0x3FFFF  # and its opposite
    want = keys[torch.argsort(keys & ((1 << bits) - 1), stable=True)]
    assert torch.equal(api.sort_u64(keys.to(DEV), bits).cpu(), want)


@pytest.mark.parametrize("n", [2, 255, 256, 257, 16383, 16384, 16385, 3 * 16384 + 1])
def test_counts_at_scan_edges(n):
    """n + 1 row offsets on both sides of one scan tile (16384), one and two vertex passes."""
    m = min(5 * n, n * (n - 1) // 2)
    rng = np.random.default_rng(n)
    a = rng.integers(0, n, 4 * m)
    b = (a + 1 + (rng.integers(0, max(n - 1, 1), 4 * m) ** 2 // max(n - 1, 1)) % max(n - 1, 1)) % n
    key = np.unique(np.minimum(a, b) * n + np.maximum(a, b))
    key = key[key // n != key % n]
    e = torch.tensor(np.stack([key // n, key % n], 1).astype(np.int32))
    want, pv = oracle.count(e, n, per_vertex=True)
    total, got = api.count_per_vertex(e.to(DEV), n)
    assert total == want == api.count(e.to(DEV), n)
    assert np.array_equal(got.cpu().numpy().astype(np.uint64), pv)
    both = torch.cat([e, e.flip(1)])[torch.randperm(2 * len(key),
                                                    generator=torch.Generator().manual_seed(n))]
    assert api.count(both.to(DEV), n, both=True) == want


def test_vertex_order_of_saturated_degrees():
    """A star and a clique: degrees up to n - 1, ranks by (degree, id)."""
    n = 300
    e = [(0, x) for x in range(1, n)] + [(i, j) for i in range(200, 260) for j in range(i + 1, 260)]
    out = api.preprocess(torch.tensor(e, dtype=torch.int32, device=DEV), n)
    deg = np.bincount(np.array(e).ravel(), minlength=n)
    assert np.array_equal(out["perm"].cpu().numpy(), np.lexsort((np.arange(n), deg)))


@pytest.mark.parametrize("m", [1, 2047, 2048, 2049, 3 * 2048])
def test_two_direction_compaction_at_tile_edges(m):
    """2 m entries on both sides of the orientation's tile (4096), forward entries first and
    last; with and without the degree partition."""
    n = m + 2
    e = torch.tensor([(x, x + 1 + (x & 1)) for x in range(m)], dtype=torch.int32)
    want = oracle.count(e, n)
    for entries in (torch.cat([e, e.flip(1)]), torch.stack([e, e.flip(1)], 1).reshape(-1, 2)):
        for part in (0, 1):
            assert api.count(entries.to(DEV), n, both=True,
                             options={"degree_partition": part}) == want
    assert api.count(e.to(DEV), n, options={"degree_partition": 0}) == want


@pytest.mark.parametrize("k", [40, 500, 723, 724, 725, 1024, 1025, 1026, 1090, 1448, 1449])
def test_rows_across_sort_chunks(k):
    """A clique's rows, of every length up to k - 1, start at all offsets of the row sort's chunks
    (512 positions below 2^18 edges, 1024 below 2^20, then 4096; rows above 1024 entries are sorted
    by another kernel) and reach into the next."""
    gen = torch.Generator().manual_seed(k)
    a, b = torch.triu_indices(k, k, 1)
    e = torch.stack([a, b], 1)[torch.randperm(a.numel(), generator=gen)].to(torch.int32)
    out = api.preprocess(e.to(DEV), k)
    col, rp = out["col"].cpu().numpy(), out["row_ptr"].cpu().numpy()
    assert np.array_equal(rp[1:] - rp[:-1], np.arange(k - 1, -1, -1))
    assert all(np.array_equal(col[rp[r]:rp[r + 1]], np.arange(r + 1, k)) for r in range(k))
    assert api.count(e.to(DEV), k) == k * (k - 1) * (k - 2) // 6


@pytest.mark.parametrize("tiles,extra", [(1, 1), (8, 0), (8, 1), (9, 1), (32, 0), (32, 1), (RAW, 1)])
@pytest.mark.parametrize("bits", [16, 34, 36, 41, 45, 49, 54, 57, 63])
def test_sort_by_ways_to_find_the_digit_starts(tiles, extra, bits):
    """Tile counts on both sides of the rules (one thread per digit up to 32 tiles, a wave per 32
    digits up to RAW, a scanned table) at the widths with digits of 9 bits above 32."""
    count = tiles * TILE + extra
    gen = torch.Generator().manual_seed(count + bits)
    keys = torch.randint(0, 1 << 62, (count,), generator=gen, dtype=torch.int64)
    keys[: count // 3] &= ~0x1FF  # a crowded digit
    keys[count // 2:] |= 0x3FFFF << 40  # and full ones
    want = keys[torch.argsort(keys & ((1 << bits) - 1), stable=True)]
    assert torch.equal(api.sort_u64(keys.to(DEV), bits).cpu(), want)
