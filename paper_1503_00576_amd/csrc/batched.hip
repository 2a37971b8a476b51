// Batched counting: many small graphs in one launch sequence, captured once in a hipGraph.
//
// Input: the graphs' symmetric adjacency lists (the format Section 3.1 contrasts with the
// edge array), concatenated.  Graph g has n_g = vtx_off[g+1] - vtx_off[g] vertices and its
// own CSR: row_ptr entries [vtx_off[g] + g, vtx_off[g+1] + g] (local offsets 0..len_g) and
// col entries [adj_off[g], adj_off[g+1]) (local ids, rows strictly ascending).  In the disjoint
// union, vertex x of graph g has id vtx_off[g] + x.
//
// Preprocessing needs no sort: the degree of a vertex is its row length, and keeping in every
// row only the neighbours that come later in the order of Section 2.2 ((degree, id)
// ascending) is a stable filter, so the oriented rows stay sorted by id.  One pass over the
// input checks it and writes every row's kept entries at the row's own place in the input:
// nothing about the other rows has to be known beforehand, so the input is read once, and a
// graph writes only inside its own adjacency range, so that a malformed one does not reach the
// others (its rows are left out when its offsets descend, or when its range meets an earlier
// graph's).  The counting kernels (count.hip) then stage N+(u) and stream N+(v) for the
// out-neighbours v.
//
// Every kernel reads the sizes and the caller's pointers from an argument block at the start
// of the workspace and runs over the plan's capacities, so one captured graph serves every
// batch that fits the plan.
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "internal.h"

namespace tc {

struct BatchArgs {
    const int64_t *vtx_off;
    const int64_t *adj_off;
    const int32_t *row_ptr;
    const int32_t *col;
    unsigned long long *totals;
    unsigned long long *per_vertex;
    int32_t *status;  // per graph, may be null
    uint32_t G, N;
    uint32_t A;  // adjacency entries in total
};

// ctl: [0] heavy-item queue, [1] heavy items, [2] first graph whose adjacency range descends (all
// ones: none, and then no two ranges meet)
enum { kCtlQueueB = 0, kCtlItemsB = 1, kCtlDescentB = 2, kCtlWordsB = 3 };

__device__ __forceinline__ void graph_error(const BatchArgs &a, uint32_t g, int32_t code,
                                            int32_t *gstat) {
    atomicCAS(&gstat[g], 0, code);
}

// graph of union vertex x: the last g with vtx_off[g] <= x
__device__ __forceinline__ uint32_t graph_of(const int64_t *vtx_off, uint32_t G, uint32_t x) {
    uint32_t lo = 0, len = G;
    while (len > 1) {
        const uint32_t half = len >> 1;
        if (vtx_off[lo + half] <= (int64_t)x) lo += half;
        len -= half;
    }
    return lo;
}

// start of a run: the argument block, zeroed outputs, statuses and counters
__global__ void k_b_begin(BatchArgs *dst, const BatchArgs a, int32_t *__restrict__ gstat,
                          unsigned long long *__restrict__ ghash, uint32_t *__restrict__ gfwd,
                          uint32_t *__restrict__ ctl) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *dst = a;
    if (i < kCtlWordsB) ctl[i] = i == kCtlDescentB ? ~0u : 0u;
    const uint32_t cap = a.per_vertex && a.N > a.G ? a.N : a.G;
    for (uint32_t x = i; x < cap; x += gridDim.x * blockDim.x) {
        if (x < a.G) {
            a.totals[x] = 0;
            gstat[x] = 0;
            ghash[x] = 0;
            gfwd[x] = 0;
        }
        if (a.per_vertex && x < a.N) a.per_vertex[x] = 0;
    }
}

// Pair hash for the symmetry check: the 64-bit finalizer of MurmurHash3 (fmix64) applied to
// (x << 32 | y).
__device__ __forceinline__ uint64_t pair_hash(uint32_t x, uint32_t y) {
    uint64_t k = ((uint64_t)x << 32) | y;
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

// per vertex: its graph, and its row length once the offsets it relies on are checked (the whole
// vertex range of its graph, whose row lengths the forward test reads).  A graph with a row whose
// offsets are bad is TC_E_ARG from here on, and k_b_setup leaves all its rows out.  per graph:
// whether its adjacency range descends
__global__ __launch_bounds__(256) void k_b_rows(const BatchArgs *__restrict__ args,
                                                uint32_t *__restrict__ gid,
                                                uint32_t *__restrict__ deg,
                                                uint32_t *__restrict__ descent,
                                                int32_t *__restrict__ gstat) {
    const BatchArgs a = *args;
    const uint32_t x = blockIdx.x * 256u + threadIdx.x;
    if (x < a.G && a.adj_off[x + 1] < a.adj_off[x]) atomicMin(descent, x);
    if (x >= a.N) return;
    uint32_t d = 0;
    const uint32_t g = graph_of(a.vtx_off, a.G, x);
    gid[x] = g;
    const int64_t v0 = a.vtx_off[g], n_g = a.vtx_off[g + 1] - v0;
    const int64_t a0 = a.adj_off[g], alen = a.adj_off[g + 1] - a0;
    const int64_t lx = (int64_t)x - v0;
    // offsets arrays must be prefix sums
    if (v0 < 0 || lx < 0 || lx >= n_g || v0 + n_g > (int64_t)a.N || a0 < 0 || alen < 0 ||
        a0 + alen > (int64_t)a.A) {
        graph_error(a, g, TC_E_ARG, gstat);
    } else {
        const int32_t *rp = a.row_ptr + v0 + g;
        const int64_t r0 = rp[lx], r1 = rp[lx + 1];
        if (r0 < 0 || r1 < r0 || r1 > alen)
            graph_error(a, g, TC_E_ARG, gstat);
        else
            d = (uint32_t)(r1 - r0);
    }
    deg[x] = d;
}

// Whether graph g's adjacency range meets that of an earlier graph with vertices (the calling wave,
// g uniform; only asked for graphs after a descent).  Ranges outside the batch hold no rows.
__device__ __forceinline__ bool meets_earlier(const BatchArgs &a, uint32_t g) {
    const int64_t b = a.adj_off[g], e = a.adj_off[g + 1];
    for (uint32_t h0 = 0; h0 < g; h0 += kWave) {
        const uint32_t h = h0 + lane_id();
        bool meets = false;
        if (h < g) {
            const int64_t hb = a.adj_off[h], he = a.adj_off[h + 1];
            meets = hb >= 0 && hb < he && he <= (int64_t)a.A && hb < e && b < he &&
                    a.vtx_off[h] < a.vtx_off[h + 1];
        }
        if (__ballot(meets)) return true;
    }
    return false;
}

// lanes a .. b - 1 of a wave (a <= b <= 64, a < 64)
__device__ __forceinline__ uint64_t lanes_from_to(uint32_t a, uint32_t b) {
    return (b >= 64 ? ~0ull : ((1ull << b) - 1ull)) & ~((1ull << a) - 1ull);
}

// The argument block's pointers are generic; the walk reads through global-address-space
// views so that its loads are global loads (waited for apart from the LDS traffic).
typedef const __attribute__((address_space(1))) int32_t *gptr_i32;

// One pass over the rows: checks (ids in range, no self-loop, strictly ascending), the forward
// rows written at the rows' places in the input, and the graph's symmetry sum and forward entries.
// (The rows of a graph that is TC_E_ARG, by k_b_rows or because its range meets an earlier graph's,
// are left out; the others are disjoint stretches of the input, so that no two rows write the same
// words and fcol and the heavy items hold them all.)
//
// A wave takes 2^vshift consecutive vertices, graph by graph (nearly always one), and walks
// their entries, consecutive in the input, 64 at a time: kWalkSteps steps together, whose loads
// are issued before any is used.  Lane l's entry belongs to row k (round_owner); the row's
// place in the input, length, first entry and output come from lane k's registers.  Rows
// run over steps, so the forward entries a row had in earlier steps are carried along (only the
// row of a step's first lane has any).
//
// Symmetry: an entry (x, y) adds the pair hash of {x, y} when it is a forward entry and takes it
// away otherwise; the two entries of an edge are forward from exactly one side, so the sum over
// a graph with symmetric rows is zero.
//
// It is bound by its vector instructions (65% of the issue slots) and the gathers of the degrees
// (64 lines a step), so every per-row value that is the same over a graph is kept in scalar
// registers, the entry before a lane's comes from its neighbour lane, one hash serves both
// directions and a degree is one 4-byte lookup.  4096 graphs of 3300 vertices (2.4e8 entries):
// 1.24 ms, where a checking pass and a second pass that wrote the rows took 1.28 + 0.65 ms.
constexpr int kWalkSteps = 4;

__global__ __launch_bounds__(256) void k_b_setup(const BatchArgs *__restrict__ args,
                                                 uint32_t vshift,
                                                 const uint32_t *__restrict__ gid,
                                                 const uint32_t *__restrict__ deg,
                                                 const uint32_t *__restrict__ descent,
                                                 uint32_t light_max, uint32_t kitem,
                                                 uint2 *__restrict__ frow,
                                                 uint32_t *__restrict__ fcol,
                                                 uint2 *__restrict__ items,
                                                 uint32_t *__restrict__ n_items,
                                                 unsigned long long *__restrict__ ghash,
                                                 uint32_t *__restrict__ gfwd,
                                                 unsigned long long *__restrict__ whash,
                                                 uint32_t *__restrict__ wfwd,
                                                 int32_t *__restrict__ gstat) {
    __shared__ uint32_t s_mark[4][kWave], s_fwd[4][kWave];
    const BatchArgs a = *args;
    const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
    uint32_t *mark = s_mark[w], *fcount = s_fwd[w];
    const uint32_t x0 = (xcd_stretch_tile(blockIdx.x, gridDim.x) * 4 + w) << vshift;
    if (x0 >= a.N) return;
    const uint32_t x = x0 + lane;
    const bool in = (lane >> vshift) == 0 && x < a.N;
    uint32_t g = ~0u, d = 0, s = 0;
    if (in) {
        g = gid[x];
        d = gstat[g] == TC_E_ARG ? 0u : deg[x];
    }
    // (no graph comes after a descent in offsets that are prefix sums)
    const uint32_t first_descent = *descent;
    for (uint64_t late = __ballot(d > 0 && g > first_descent); late;) {
        const uint32_t gc = (uint32_t)__builtin_amdgcn_readlane((int)g, __ffsll((long long)late) - 1);
        late &= ~__ballot(g == gc);
        if (!meets_earlier(a, gc)) continue;
        if (g == gc) {
            graph_error(a, g, TC_E_ARG, gstat);
            d = 0;
        }
    }
    mark[lane] = 0;
    fcount[lane] = 0;
    const gptr_i32 col = (gptr_i32)a.col;
    uint32_t round = 0;
    uint64_t part_h = 0;  // lanes 0 and 1: this wave's parts of graphs that span waves
    uint32_t part_f = 0;
    for (uint64_t todo = __ballot(d > 0); todo;) {
        const uint32_t gc = (uint32_t)__builtin_amdgcn_readlane((int)g, __ffsll((long long)todo) - 1);
        const bool mine = d > 0 && g == gc;
        todo &= ~__ballot(mine);
        const int64_t v0 = a.vtx_off[gc];
        const uint32_t ng = (uint32_t)(a.vtx_off[gc + 1] - v0);
        const gptr_i32 rp = (gptr_i32)(a.row_ptr + v0 + gc);
        const gptr_i32 gdeg = (gptr_i32)(deg + v0);
        const uint32_t lx0 = x0 - (uint32_t)v0;  // local id of lane 0's vertex (modulo 2^32)
        const uint32_t dm = mine ? d : 0u;
        const uint32_t incl = wave_incl_scan(dm), off = incl - dm;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        if (mine) s = (uint32_t)(a.adj_off[gc] + rp[(uint32_t)(lx0 + lane)]);
        const uint32_t in_at = s - off;  // the row's place in the input, less its place in the walk
        uint32_t carry = 0, carry_f = 0;
        int32_t y_last = -1;
        uint64_t hsum = 0;
        // kWalkSteps steps from `base` on; full: every lane has an entry in each.  Conditions are
        // combined without short circuits, so that a step has no branch but the stores'.
        auto walk = [&](uint32_t base, auto full) {
            uint32_t k[kWalkSteps];
            int32_t y[kWalkSteps], dy[kWalkSteps];
#pragma unroll
            for (int u = 0; u < kWalkSteps; ++u) {
                k[u] = round_owner(mark, off, dm, base + u * kWave, ++round, carry) - 1u;
                const uint32_t at = wave_bcast_from(in_at, k[u]);
                const uint32_t idx = base + u * kWave + lane;
                y[u] = (full || idx < total) ? col[at + idx] : 0;
            }
#pragma unroll
            for (int u = 0; u < kWalkSteps; ++u)
                dy[u] = gdeg[(uint32_t)y[u] < ng ? (uint32_t)y[u] : 0u];
#pragma unroll
            for (int u = 0; u < kWalkSteps; ++u) {
                const uint32_t sb = base + u * kWave, idx = sb + lane;
                const bool valid = full || idx < total;
                const uint32_t dk = wave_bcast_from(d, k[u]), ok_ = wave_bcast_from(off, k[u]);
                const uint32_t sk = wave_bcast_from(s, k[u]);
                const uint32_t yu = (uint32_t)y[u], lk = valid ? lx0 + k[u] : 0u;
                const bool ok = (yu < ng) & (yu != lk) & valid;
                const bool fwd =
                    ok & ((dy[u] > (int32_t)dk) | ((dy[u] == (int32_t)dk) & (yu > lk)));
                // the entry before this one (lane 0: the previous step's last)
                const int32_t prev = __builtin_amdgcn_update_dpp(y_last, y[u], 0x138, 0xf, 0xf,
                                                                 false);  // wave_shr:1
                y_last = __builtin_amdgcn_readlane(y[u], kWave - 1);
                const bool bad = valid & (!ok | ((idx > ok_) & (y[u] <= prev)));
                if (__ballot(bad)) {
                    if (bad)
                        graph_error(a, gc,
                                    !ok ? (yu >= ng ? TC_E_RANGE : TC_E_SELF_LOOP)
                                        : (y[u] == prev ? TC_E_DUP_EDGE : TC_E_UNSORTED),
                                    gstat);
                }
                // (lanes without an entry hash the pair {0, 0} to 0; a graph with other entries
                // that are not ok is reported whatever its sum)
                const uint64_t h = pair_hash(min(lk, yu), max(lk, yu));
                hsum += fwd ? h : 0ull - h;
                // forward entries of the row before this one.  (`& 63u` changes nothing where the row
                // starts in this step.  It has to be there, and not as min(.., 63u): with that the
                // compiler, clang 20 of ROCm 7.2, took `begun` for true in all steps, and rows that
                // run over steps lost what carry_f holds.  test_light_rows_at_window_edges and
                // test_batched_one_shot have such rows.)
                const uint64_t F = __ballot(fwd);
                const bool begun = ok_ >= sb;  // the row starts in this step
                const uint32_t rank = (uint32_t)__popcll(
                    F & lanes_from_to(begun ? (ok_ - sb) & 63u : 0u, lane)) + (begun ? 0u : carry_f);
                if (fwd) fcol[sk + rank] = (uint32_t)v0 + yu;
                const uint32_t upto = rank + (fwd ? 1u : 0u);
                if (valid & (idx + 1 == ok_ + dk)) fcount[k[u]] = upto;
                carry_f = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
            }
        };
        uint32_t base = 0;
        for (; base + kWalkSteps * kWave <= total; base += kWalkSteps * kWave)
            walk(base, std::true_type{});
        if (base < total) walk(base, std::false_type{});
        wave_lds_sync();
        const uint64_t hs = wave_sum_u64(hsum);
        const uint32_t fs = wave_total(mine ? fcount[lane] : 0u);
        const uint32_t span = graph_span(a.vtx_off, gc, x0, vshift);
        if (span == kSpanWhole) {
            if (lane == 0) {
                ghash[gc] = hs;
                gfwd[gc] = fs;
            }
        } else if (lane == span) {
            part_h = hs;
            part_f = fs;
        }
    }
    if (lane < 2) {
        whash[2 * (x0 >> vshift) + lane] = part_h;
        wfwd[2 * (x0 >> vshift) + lane] = part_f;
    }
    const uint32_t f = d > 0 ? fcount[lane] : 0u;
    if (in) frow[x] = make_uint2(s, s + f);
    // heavy rows (more than light_max forward neighbours) in items of kitem of them
    const uint32_t ni = f > light_max ? (f + kitem - 1) / kitem : 0u;
    if (__ballot(ni > 0)) {
        const uint32_t iincl = wave_incl_scan(ni);
        uint32_t at = 0;
        if (lane == kWave - 1) at = atomicAdd(n_items, iincl);
        at = wave_bcast(at, kWave - 1) + iincl - ni;
        for (uint32_t j = 0; j < ni; ++j) items[at + j] = make_uint2(x, s + j * kitem);
    }
}

// one wave per graph: the sums of a graph that spans waves from their parts, the checks that
// need the whole graph, and the status out (the caller's array, when given).  Offsets: the
// graph's vertex and adjacency ranges must lie inside the batch (k_b_rows checked them only for
// graphs that have vertices).  Symmetry: the entries must number twice the forward entries, and
// the graph's symmetry sum must be zero (a set of entries that is not closed under mirroring
// passes this with probability about 2^-64).
__global__ __launch_bounds__(256) void k_b_finish(const BatchArgs *__restrict__ args,
                                                  uint32_t vshift,
                                                  const unsigned long long *__restrict__ ghash,
                                                  const uint32_t *__restrict__ gfwd,
                                                  const unsigned long long *__restrict__ whash,
                                                  const uint32_t *__restrict__ wfwd,
                                                  const unsigned long long *__restrict__ wtotal,
                                                  const int32_t *__restrict__ gstat) {
    const BatchArgs a = *args;
    const uint32_t g = blockIdx.x * 4 + threadIdx.x / kWave, lane = lane_id();
    if (g >= a.G) return;
    const int64_t v0 = a.vtx_off[g], v1 = a.vtx_off[g + 1];
    const int64_t a0 = a.adj_off[g], a1 = a.adj_off[g + 1];
    int32_t st = gstat[g];
    const bool inside = v0 >= 0 && v1 >= v0 && v1 <= (int64_t)a.N && a0 >= 0 && a1 >= a0 &&
                        a1 <= (int64_t)a.A;
    if (st == 0 && !inside) st = TC_E_ARG;
    if (inside) {
        uint64_t h = 0, t = 0, f = 0;
        const uint32_t w0 = (uint32_t)v0 >> vshift;
        if (v1 > v0 && ((uint32_t)(v1 - 1) >> vshift) > w0) {
            const uint32_t w1 = (uint32_t)(v1 - 1) >> vshift;
            for (uint32_t w = w0 + lane; w <= w1; w += kWave) {
                const uint32_t i = 2 * w + (w == w0 ? kSpanAfter : kSpanBefore);
                h += whash[i];
                f += wfwd[i];
                t += wtotal[i];
            }
            h = wave_sum_u64(h);
            f = wave_sum_u64(f);
            t = wave_sum_u64(t);
            if (lane == 0 && t) a.totals[g] += t;
        } else {
            h = ghash[g];
            f = gfwd[g];
        }
        if (st == 0 && (2 * (int64_t)f != a1 - a0 || h != 0)) st = TC_E_ASYMMETRIC;
    }
    if (a.status && lane == 0) a.status[g] = st;
}

// ------------------------------------------------------------------ workspace + plan

struct BatchLayout {
    size_t args, ctl, gstat, ghash, gfwd, gid, deg, frow, fcol, items, whash, wfwd, wtotal,
        total;
};

constexpr uint32_t kMinItemEdges = 16;

// Vertices per wave of the setup and the light counting: 64, or fewer when that leaves the chip
// idle (down to 8, below 8192 waves: eight for each of the 1024 SIMDs, what they hold at most).  Counting four R-MAT graphs of 15,360 vertices
// together took 950 us when 38 waves shared them and takes 59 us with 1920.
static uint32_t batch_vshift(uint32_t ncap) {
    uint32_t v = 6;
    while (v > 3 && (ncap >> v) < 8192u) --v;
    return v;
}

}  // namespace tc

using namespace tc;

struct tc_plan {
    uint32_t gcap, ncap;
    uint64_t acap;
    uint32_t kitem, chunk, wgs_per_cu;
    uint32_t light_max;  // forward-degree threshold of the edge-per-lane path
    uint32_t wave_bits;  // heavy items: bitmap below this id span
    uint32_t wave_list;  // heavy items: sorted LDS list of at most this many entries
    void *ws;
    size_t ws_bytes;
    BatchLayout L;
    hipGraph_t graph[2];
    hipGraphExec_t exec[2];
};

static uint32_t parse_tuning(const char *json, const char *key, uint32_t dflt) {
    if (!json) return dflt;
    const char *p = strstr(json, key);
    if (!p) return dflt;
    p = strchr(p + strlen(key), ':');
    if (!p) return dflt;
    long v = strtol(p + 1, nullptr, 10);
    return v > 0 ? (uint32_t)v : dflt;
}

// as parse_tuning, but 0 is a value (negative values give the default)
static uint32_t parse_tuning_or_zero(const char *json, const char *key, uint32_t dflt) {
    if (!json) return dflt;
    const char *p = strstr(json, key);
    if (!p) return dflt;
    p = strchr(p + strlen(key), ':');
    if (!p) return dflt;
    long v = strtol(p + 1, nullptr, 10);
    return v >= 0 ? (uint32_t)(v > 0x7FFFFFFFl ? 0x7FFFFFFFl : v) : dflt;
}

static BatchLayout batch_layout(uint32_t gcap, uint32_t ncap, uint64_t acap) {
    BatchLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off = align_up(off + (bytes ? bytes : 1), 256);
        return at;
    };
    L.args = take(sizeof(BatchArgs));
    L.ctl = take(64 * 4);
    L.gstat = take((size_t)gcap * 4);
    L.ghash = take((size_t)gcap * 8);
    L.gfwd = take((size_t)gcap * 4);
    L.gid = take((size_t)ncap * 4);
    L.deg = take((size_t)ncap * 4);
    L.frow = take((size_t)ncap * 8);
    L.fcol = take((size_t)acap * 4 + count_col_pad_bytes());
    L.items = take(((size_t)acap / kMinItemEdges + ncap + 1) * 8);
    const size_t parts = 2 * (((size_t)ncap >> batch_vshift(ncap)) + 1);
    L.whash = take(parts * 8);
    L.wfwd = take(parts * 4);
    L.wtotal = take(parts * 8);
    L.total = off;
    return L;
}

// enqueue the whole sequence after k_b_begin (this is what gets captured)
static int batch_enqueue(tc_plan *p, bool pv, hipStream_t s) {
    const BatchLayout &L = p->L;
    char *ws = (char *)p->ws;
    const BatchArgs *args = (const BatchArgs *)(ws + L.args);
    uint32_t *ctl = (uint32_t *)(ws + L.ctl);
    int32_t *gstat = (int32_t *)(ws + L.gstat);
    unsigned long long *ghash = (unsigned long long *)(ws + L.ghash);
    unsigned long long *whash = (unsigned long long *)(ws + L.whash);
    unsigned long long *wtotal = (unsigned long long *)(ws + L.wtotal);
    uint32_t *gfwd = (uint32_t *)(ws + L.gfwd), *wfwd = (uint32_t *)(ws + L.wfwd);
    uint32_t *gid = (uint32_t *)(ws + L.gid), *deg = (uint32_t *)(ws + L.deg);
    uint32_t *fcol = (uint32_t *)(ws + L.fcol);
    uint2 *frow = (uint2 *)(ws + L.frow), *items = (uint2 *)(ws + L.items);
    const uint32_t ncap = p->ncap, vshift = batch_vshift(ncap);
    const uint32_t rows = ncap > p->gcap ? ncap : p->gcap;
    hipLaunchKernelGGL(k_b_rows, dim3(ceil_div(rows, 256)), dim3(256), 0, s, args, gid, deg,
                       ctl + kCtlDescentB, gstat);
    if (hipGetLastError() != hipSuccess) return TC_E_HIP;
    const uint32_t waves = ceil_div(ncap > 0 ? ncap : 1, 1ull << vshift);
    hipLaunchKernelGGL(k_b_setup, dim3(ceil_div(waves, 4)), dim3(256), 0, s, args,
                       vshift, gid, deg, ctl + kCtlDescentB, p->light_max, p->kitem, frow, fcol,
                       items, ctl + kCtlItemsB, ghash, gfwd, whash, wfwd, gstat);
    if (hipGetLastError() != hipSuccess) return TC_E_HIP;
    BatchKernelArgs ka;
    ka.frow = frow;
    ka.fcol = fcol;
    ka.gid = gid;
    ka.items = items;
    ka.n_items = ctl + kCtlItemsB;
    ka.n = &args->N;
    ka.vtx_off_pp = &args->vtx_off;
    ka.wtotal = wtotal;
    ka.queue = ctl + kCtlQueueB;
    ka.totals_pp = &args->totals;
    ka.tpv_pp = &args->per_vertex;
    ka.kitem = p->kitem;
    ka.light_max = p->light_max;
    ka.wave_bits = p->wave_bits;
    ka.wave_list = pv ? (p->wave_list < count_wave_list(true) ? p->wave_list
                                                              : count_wave_list(true))
                      : p->wave_list;
    ka.window = count_light_window(p->chunk, p->light_max);
    if (launch_count_u(ka, pv, device_cu_count() * p->wgs_per_cu, ncap, vshift, s) != hipSuccess)
        return TC_E_HIP;
    hipLaunchKernelGGL(k_b_finish, dim3(ceil_div(p->gcap, 4)), dim3(256), 0, s, args, vshift,
                       ghash, gfwd, whash, wfwd, wtotal, gstat);
    return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

static int batch_capture(tc_plan *p, bool pv) {
    const int k = pv ? 1 : 0;
    if (p->exec[k]) return TC_OK;
    hipStream_t cs;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return TC_E_HIP;
    int st = TC_OK;
    if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        (void)hipStreamDestroy(cs);
        return TC_E_HIP;
    }
    st = batch_enqueue(p, pv, cs);
    hipGraph_t g = nullptr;
    if (hipStreamEndCapture(cs, &g) != hipSuccess || !g) st = TC_E_HIP;
    (void)hipStreamDestroy(cs);
    if (st != TC_OK) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    hipGraphExec_t ex = nullptr;
    if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGraphDestroy(g);
        return TC_E_HIP;
    }
    p->graph[k] = g;
    p->exec[k] = ex;
    return TC_OK;
}

static int plan_set_args(tc_plan *p, int32_t G, const int64_t *d_vtx_off,
                         const int64_t *d_adj_off, const int32_t *d_row_ptr,
                         const int32_t *d_col, int64_t n_total, int64_t adj_total,
                         hipStream_t s, uint64_t *d_totals, uint64_t *d_per_vertex,
                         int32_t *d_status) {
    if (G <= 0 || !d_vtx_off || !d_adj_off || !d_row_ptr || !d_totals) return TC_E_ARG;
    if ((uint32_t)G > p->gcap || n_total < 0 || (uint64_t)n_total > p->ncap || adj_total < 0 ||
        (uint64_t)adj_total > p->acap)
        return TC_E_TOO_LARGE;
    if (adj_total > 0 && !d_col) return TC_E_ARG;
    BatchArgs a;
    a.vtx_off = d_vtx_off;
    a.adj_off = d_adj_off;
    a.row_ptr = d_row_ptr;
    a.col = d_col;
    a.totals = (unsigned long long *)d_totals;
    a.per_vertex = (unsigned long long *)d_per_vertex;
    a.status = d_status;
    a.G = (uint32_t)G;
    a.N = (uint32_t)n_total;
    a.A = (uint32_t)adj_total;
    char *ws = (char *)p->ws;
    const uint64_t cap = d_per_vertex && n_total > G ? (uint64_t)n_total : (uint64_t)G;
    const uint32_t blocks = ceil_div(cap, 256) < 1024u ? ceil_div(cap, 256) : 1024u;
    hipLaunchKernelGGL(k_b_begin, dim3(blocks), dim3(256), 0, s, (BatchArgs *)(ws + p->L.args), a,
                       (int32_t *)(ws + p->L.gstat), (unsigned long long *)(ws + p->L.ghash),
                       (uint32_t *)(ws + p->L.gfwd), (uint32_t *)(ws + p->L.ctl));
    return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

extern "C" {

size_t tc_batched_workspace_size(int32_t g_cap, int64_t n_cap, int64_t adj_cap) {
    if (g_cap <= 0 || n_cap < 0 || adj_cap < 0 || n_cap >= (1ll << 31) ||
        adj_cap >= (1ll << 32))
        return 0;
    return batch_layout((uint32_t)g_cap, (uint32_t)n_cap, (uint64_t)adj_cap).total;
}

int tc_batched_plan_create(int32_t g_cap, int64_t n_cap, int64_t adj_cap, uint32_t flags,
                           const char *tuning_json, void *d_ws, size_t ws_bytes,
                           tc_plan **out) {
    if (!out) return TC_E_ARG;
    *out = nullptr;
    if (g_cap <= 0 || n_cap < 0 || adj_cap < 0 || flags != 0) return TC_E_ARG;
    if (n_cap >= (1ll << 31) || adj_cap >= (1ll << 32)) return TC_E_TOO_LARGE;
    const BatchLayout L = batch_layout((uint32_t)g_cap, (uint32_t)n_cap, (uint64_t)adj_cap);
    if (!d_ws || ((uintptr_t)d_ws & 255) || ws_bytes < L.total) return TC_E_WORKSPACE;
    tc_plan *p = (tc_plan *)calloc(1, sizeof(tc_plan));
    if (!p) return TC_E_ARG;
    p->gcap = (uint32_t)g_cap;
    p->ncap = (uint32_t)n_cap;
    p->acap = (uint64_t)adj_cap;
    p->kitem = parse_tuning(tuning_json, "\"items_k\"", 256);
    if (p->kitem < kMinItemEdges) p->kitem = kMinItemEdges;
    p->chunk = parse_tuning(tuning_json, "\"chunk_e\"", 1024);
    if (p->chunk < 64) p->chunk = 64;
    if (p->chunk > count_light_chunk_max()) p->chunk = count_light_chunk_max();
    p->wgs_per_cu = parse_tuning(tuning_json, "\"wgs_per_cu\"", count_wgs_per_cu());
    if (p->wgs_per_cu > count_wgs_per_cu()) p->wgs_per_cu = count_wgs_per_cu();  // LDS limit
    // the light/heavy threshold and the heavy items' LDS forms: the defaults are the largest
    // values the LDS holds; lower values are accepted (tuning, and tests that reach every
    // form on small graphs)
    p->light_max = parse_tuning_or_zero(tuning_json, "\"light_max\"", count_light_max());
    if (p->light_max > count_light_max()) p->light_max = count_light_max();
    p->wave_bits = parse_tuning_or_zero(tuning_json, "\"bitmap_span\"", count_wave_span());
    if (p->wave_bits > count_wave_span()) p->wave_bits = count_wave_span();
    p->wave_list = parse_tuning_or_zero(tuning_json, "\"list_max\"", count_wave_list(false));
    if (p->wave_list > count_wave_list(false)) p->wave_list = count_wave_list(false);
    p->ws = d_ws;
    p->ws_bytes = ws_bytes;
    p->L = L;
    *out = p;
    return TC_OK;
}

int tc_batched_plan_run(tc_plan *p, int32_t G, const int64_t *d_vtx_off,
                        const int64_t *d_adj_off, const int32_t *d_row_ptr, const int32_t *d_col,
                        int64_t n_total, int64_t adj_total, void *stream, uint64_t *d_totals,
                        uint64_t *d_per_vertex, int32_t *d_status) {
    if (!p) return TC_E_ARG;
    const bool pv = d_per_vertex != nullptr;
    int st = batch_capture(p, pv);
    if (st) return st;
    hipStream_t s = (hipStream_t)stream;
    st = plan_set_args(p, G, d_vtx_off, d_adj_off, d_row_ptr, d_col, n_total, adj_total, s,
                       d_totals, d_per_vertex, d_status);
    if (st) return st;
    if (hipGraphLaunch(p->exec[pv ? 1 : 0], s) != hipSuccess) return TC_E_HIP;
    return TC_OK;
}

void tc_batched_plan_destroy(tc_plan *p) {
    if (!p) return;
    for (int k = 0; k < 2; ++k) {
        if (p->exec[k]) (void)hipGraphExecDestroy(p->exec[k]);
        if (p->graph[k]) (void)hipGraphDestroy(p->graph[k]);
    }
    free(p);
}

int tc_count_batched(int32_t G, const int64_t *d_vtx_off, const int64_t *d_adj_off,
                     const int32_t *d_row_ptr, const int32_t *d_col, int64_t n_total,
                     int64_t adj_total, void *d_ws, size_t ws_bytes, void *stream,
                     uint64_t *d_totals, uint64_t *d_per_vertex, int32_t *d_status) {
    tc_plan *p = nullptr;
    int st = tc_batched_plan_create(G, n_total, adj_total, 0, nullptr, d_ws, ws_bytes, &p);
    if (st) return st;
    st = plan_set_args(p, G, d_vtx_off, d_adj_off, d_row_ptr, d_col, n_total, adj_total,
                       (hipStream_t)stream, d_totals, d_per_vertex, d_status);
    if (st == TC_OK) st = batch_enqueue(p, d_per_vertex != nullptr, (hipStream_t)stream);
    tc_batched_plan_destroy(p);
    return st;
}

}  // extern "C"
