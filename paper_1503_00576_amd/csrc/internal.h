// Internal declarations shared by the HIP translation units of libtc.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/tc.h"

namespace tc {

constexpr int kWave = 64;

// ---------------------------------------------------------------- device helpers

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// number of set bits of `mask` at lanes below the calling lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Orders this wave's LDS accesses before the ones that follow (all lanes of a wave).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t wave_bcast(uint32_t x, int src) {
    return (uint32_t)__shfl((int)x, src, kWave);
}

// x of lane src (a per-lane index; all lanes active)
__device__ __forceinline__ uint32_t wave_bcast_from(uint32_t x, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)x);
}

// inclusive prefix sum over the 64 lanes (all lanes active): row shifts by 1, 2, 4, 8 inside each
// 16-lane row (lanes shifted in from outside read 0), then the last lane of rows 0 and 2 into
// rows 1 and 3, and lane 31 into rows 2 and 3; six vector adds, where shuffles through the LDS
// crossbar cost six round trips of it
template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_add_step(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRowMask, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v = dpp_add_step<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add_step<0x112, 0xf>(v);  // row_shr:2
    v = dpp_add_step<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add_step<0x118, 0xf>(v);  // row_shr:8
    v = dpp_add_step<0x142, 0xa>(v);  // row_bcast:15
    v = dpp_add_step<0x143, 0xc>(v);  // row_bcast:31
    return v;
}

// inclusive prefix maximum over the 64 lanes (all lanes active): row shifts by 1, 2, 4, 8
// inside each 16-lane row (lanes shifted in from outside read 0), then the last lane of rows
// 0 and 2 into rows 1 and 3, and lane 31 into rows 2 and 3
template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_max_step(uint32_t v) {
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRowMask, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v) {
    v = dpp_max_step<0x111, 0xf>(v);  // row_shr:1
    v = dpp_max_step<0x112, 0xf>(v);  // row_shr:2
    v = dpp_max_step<0x114, 0xf>(v);  // row_shr:4
    v = dpp_max_step<0x118, 0xf>(v);  // row_shr:8
    v = dpp_max_step<0x142, 0xa>(v);  // row_bcast:15
    v = dpp_max_step<0x143, 0xc>(v);  // row_bcast:31
    return v;
}

__device__ __forceinline__ uint32_t wave_total(uint32_t x) {  // sum over the lanes, in all lanes
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(x), kWave - 1);
}

// Owner of element base + lane of a sequence cut into runs, one run per lane: every run whose
// start (my_off, of this lane's run, non-empty when `any`) falls in the 64 elements from base on
// marks that lane in the wave's table (tagged with the round number, so older marks read as
// none; rounds count from 1, the table cleared beforehand), and the running maximum over the
// lanes carries the last mark forward; lanes before the round's first mark belong to carry, the
// previous round's last run (plus one).  Returns the owner plus one (all lanes active).
__device__ __forceinline__ uint32_t round_owner(uint32_t *mark, uint32_t my_off, uint32_t any,
                                                uint32_t base, uint32_t round, uint32_t &carry) {
    const uint32_t lane = lane_id();
    const uint32_t pos = my_off - base;
    if (any && pos < kWave) mark[pos] = (round << 7) | (lane + 1u);
    wave_lds_sync();
    const uint32_t mv = mark[lane];
    const uint32_t m1 = wave_incl_max((mv >> 7) == round ? (mv & 127u) : 0u);
    const uint32_t owner1 = m1 ? m1 : carry;
    carry = (uint32_t)__builtin_amdgcn_readlane((int)owner1, kWave - 1);
    return owner1;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, d, kWave);
        uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), d, kWave);
        x += ((uint64_t)hi << 32) | lo;
    }
    return x;
}

__device__ __forceinline__ void set_status(int32_t *st, int32_t code) {
    atomicCAS(st, 0, code);
}

// ---------------------------------------------------------------- host helpers

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline uint32_t ceil_div(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// Workgroups are dispatched round-robin over the chip's 8 XCDs, each with its own L2.  Tiled
// kernels whose neighbouring tiles share cache lines (per-tile tables stored tile-minor) map
// workgroup b of nb to tile xcd_tile(b, nb), so that every XCD works through one contiguous
// range of tiles.  A bijection of [0, nb).
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t nb) {
    const uint32_t x = b % kXcds, i = b / kXcds, q = nb / kXcds, r = nb % kXcds;
    return x * q + (x < r ? x : r) + i;
}

// The same in stretches of 64 tiles per XCD, so that a grid whose tiles differ in work stays
// balanced over the XCDs (the tiles after the last full set of stretches keep their places).
constexpr uint32_t kXcdStretch = 64;
__device__ __forceinline__ uint32_t xcd_stretch_tile(uint32_t b, uint32_t nb) {
    constexpr uint32_t set = kXcds * kXcdStretch;
    if (b >= nb / set * set) return b;
    const uint32_t i = b % set;
    return b - i + (i % kXcds) * kXcdStretch + i / kXcds;
}

// exclusive scans of uint32; scratch: scan_scratch_words(N) words.  Of an array (in may equal
// out), of four at once, of row lengths from the rows' bounds, of the rows' room in hcol (the
// last two also write out[rows], the total)
size_t scan_scratch_words(uint64_t N);
hipError_t scan_four_u32(uint32_t *const in[4], uint32_t *const out[4], uint64_t N,
                         uint32_t *scratch, hipStream_t s);
hipError_t scan_row_bounds(const uint32_t *rs, const uint32_t *re, uint64_t rows, uint32_t *out,
                           uint32_t *scratch, hipStream_t s);
hipError_t scan_high_rows(const uint32_t *row_ptr, const uint32_t *hrow, uint64_t rows,
                          uint32_t pad, uint32_t *out, uint32_t *scratch, hipStream_t s);
hipError_t scan_exclusive_u32(const uint32_t *in, uint32_t *out, uint64_t N, uint32_t *scratch,
                              hipStream_t s);

// radix sort: result lands in *result (== keys or tmp); scratch: sort_scratch_bytes(count);
// onesweep: single-sweep passes for sorts of at least 2^20 keys (needs a status word)
size_t sort_scratch_bytes(uint64_t count);
hipError_t sort_u64(uint64_t *keys, uint64_t *tmp, uint32_t count, int lo_bit, int hi_bit,
                    void *scratch, int32_t *status, hipStream_t s, uint64_t **result,
                    bool onesweep = false);
// keys sorted (stably) on bits lo_bit .. hi_bit and written unzipped: col[i] = low b bits,
// src[i] = the bits above (keys and tmp are clobbered); same scratch as sort_u64
hipError_t sort_unzip(uint64_t *keys, uint64_t *tmp, uint32_t count, int lo_bit, int hi_bit,
                      int b, uint32_t *col, uint32_t *src, void *scratch, int32_t *status,
                      hipStream_t s, bool onesweep = false);
// the vertex order: the ids 0 .. n - 1 sorted (stably) by degree (below 2^b; larger ones, which
// only invalid input has, are cut off), the last pass writing perm[r] = id of position r and
// rank[id] = r; keys and tmp: n keys of room each; same scratch as sort_u64
hipError_t sort_ranks(const uint32_t *deg, uint64_t *keys, uint64_t *tmp, uint32_t n, int b,
                      uint32_t *perm, uint32_t *rank, void *scratch, int32_t *status,
                      hipStream_t s);
// The in-edge lists: the keys (cid[i] << 32) | i with cid[i] != drop sorted (stably) on their
// bits 32 .. 32 + bits, written split: *list (list ids, in a or b, whichever the last pass
// does not read) and cbeg (position + 1), *kept of them (a device word).  The first pass
// reads the 32-bit ids and drops the others, the middle ones ping-pong between a and b on the
// kept keys (cid may alias b, not a); two-kernel passes; same scratch as sort_u64.
hipError_t sort_lists(const uint32_t *cid, uint32_t drop, uint32_t count, int bits,
                      uint64_t *a, uint64_t *b, uint32_t *cbeg, uint32_t *kept, void *scratch,
                      int32_t *status, hipStream_t s, uint32_t **list);

// arrays filled by one launch (16-byte aligned)
struct Fill {
    uint32_t *p;
    uint64_t words;
    uint32_t value;
};
struct FillList {
    Fill a[13];
    int count = 0;
    void add(uint32_t *p, uint32_t value, uint64_t words) {
        if (words) a[count++] = Fill{p, words, value};
    }
};
hipError_t fill_all(const FillList &f, hipStream_t s);
hipError_t fill_u32(uint32_t *p, uint32_t value, uint64_t count, hipStream_t s);

// preprocessing of small graphs (small.hip): at most small_vertices() vertices, small_entries()
// entries.  Degrees (deg cleared) and order; rows (re and counter cleared, rs zero) in any order
// inside, with rchunk for the row sort; in-edge lists from the in-edges' list ids (lre cleared, lrs
// zero; lre[c] = the entries of list c)
uint32_t small_vertices();
uint32_t small_entries();
hipError_t small_order(const int32_t *edges, uint32_t m, uint32_t n, bool both, uint32_t *deg,
                       uint32_t *perm, uint32_t *rank, int32_t *status, hipStream_t s);
hipError_t small_rows(const int32_t *edges, uint32_t m, uint32_t n, bool both, uint32_t mf,
                      const uint32_t *rank, uint2 *tmp, const uint32_t *rs, uint32_t *re,
                      uint32_t *row_ptr, uint32_t *col, uint32_t *src, uint32_t *rchunk,
                      uint32_t *counter, uint32_t *scan_scratch, int32_t *status, hipStream_t s);
hipError_t small_lists(const uint32_t *cid, uint32_t mf, uint32_t lists, const uint32_t *lrs,
                       uint32_t *lre, uint32_t *pos, uint32_t *cptr, uint32_t *cbeg,
                       uint32_t *scan_scratch, int32_t *status, hipStream_t s);

int device_cu_count();

// the work items' four queues: wave / workgroup items of totals, then of per-vertex counts; list c
// has items[k][c] items, the first at list[k][off[k][c]]
struct ItemLists {
    uint32_t *items[4], *off[4], *list[4];
};

// counting kernels (count.hip)
struct CountArgs {
    // in-edge lists: entry j of list c (cptr[c] <= j < cptr[c + 1]) is the in-edge at CSR
    // position cbeg[j] - 1, whose record er[cbeg[j] - 1] = (end of its row, panel mask or where
    // the suffix's entries >= hbase start in col, where they start in hcol, its row)
    const uint32_t *row_ptr, *col, *cptr, *cbeg;
    const uint4 *er;
    // every row's entries >= rank hbase as 16-bit offsets from hbase, each row's part 8-aligned
    // and followed by zeros (count_hcol_pad()); totals stream every in-edge suffix's entries
    // >= hbase from here
    const uint16_t *hcol;
    const uint32_t *hrow;  // first position >= hbase of every row, all ones for none
    uint32_t hbase;        // n: no high region
    const uint32_t *item_v_a, *item_off_a, *n_items_a;
    const uint32_t *item_v_b, *item_off_b, *n_items_b;
    uint32_t *queue_a, *queue_b;
    uint32_t *queue_c;  // per-vertex counts: the panels of k_count_panel_pv
    unsigned long long *total, *tpv;
    uint32_t n1;
    uint32_t p0;          // first rank of the panel region (n: no panels)
    const uint32_t *first_panel;  // first rank counted in panels (from p0 on; k_panel_range)
    uint32_t wave_bits;   // wave items use a bitmap below this rank span
    uint32_t block_bits;  // workgroup items use a bitmap below this rank span (totals)
    uint32_t block_list;  // ... else an LDS list of at most this many entries (<= kBlockList)
    uint32_t kitem_a;     // in-edges per wave item
    uint32_t kitem_b;     // in-edges per workgroup item
    uint32_t lists;       // in-edge lists in all
    uint32_t light;       // lists of at most this many in-edges and entries of N+(v) are light
                          // (0: none); k_items gives them no items
    unsigned long long *light_total;  // kLightTotals counters a cache line apart, cleared
    const int32_t *status;
};
constexpr uint32_t kLightTotals = 64, kLightTotalStep = 16;
uint32_t count_light_list();  // the largest light list
hipError_t launch_count(const CountArgs &a, bool per_vertex, hipStream_t s);
// LDS limits of the counting kernels' per-item structures (the defaults of the options)
uint32_t count_wave_span();         // wave bitmap: rank span below this
uint32_t count_wave_list(bool per_vertex);   // wave sorted list: entries
uint32_t count_block_span();        // workgroup bitmap: rank span below this
uint32_t count_block_list(bool per_vertex);  // workgroup sorted list: entries
uint32_t count_item_edges_wave();   // default in-edges per wave item
uint32_t count_item_edges_block();  // default in-edges per workgroup item
// bytes of padding `col` needs after its last element: a lane's aligned piece reads may run
// up to one piece past the end of a list
uint32_t count_col_pad_bytes();
// the per-row sort after a sort of the edge keys by source only: CSR positions per chunk
// (k_row_sort's workgroups), and the longest row one wave sorts (longer rows are listed)
uint32_t row_sort_chunk(uint64_t mf);
uint32_t row_sort_wave();
// zeros after every row's part of hcol beyond its rounding to 8 entries (a piece of the
// unmasked probes read from an 8-aligned position inside the part never leaves it)
uint32_t count_hcol_pad();
// middle-vertex panels: consecutive ranks per panel, and the largest rank region the
// counting kernel can handle as panels (its mask table must fit the workgroup's LDS)
uint32_t count_panel();
uint32_t count_wgs_per_cu();  // resident workgroups per CU of the counting kernels
uint32_t count_panel_ranks();
// hub triangles on the matrix cores (hub.hip): A / At are hp x hp int8, hubs = ranks h0 ..
hipError_t launch_hub_fill(const uint32_t *src, const uint32_t *col, const uint32_t *row_ptr,
                           uint32_t mf, uint32_t h0, uint32_t hp, uint8_t *A, uint8_t *At,
                           const int32_t *status, hipStream_t s);
hipError_t launch_hub_count(const uint8_t *A, const uint8_t *At, uint32_t hp, uint32_t h0,
                            unsigned long long *total, unsigned long long *tpv, bool per_vertex,
                            const int32_t *status, hipStream_t s);
// A wave's sums for the graphs of its vertices.  A graph that lies in one wave's vertices gets its
// sum directly; one that spans waves has a part from each, without atomics (the waves of a graph
// run together and would queue on its address, 11 ns each: 36 us for 1920 waves of four graphs):
// wave w keeps the part of the graph that began before its vertices at entry 2 w, the part of the
// graph that begins in them and goes on at entry 2 w + 1.  k_b_finish adds them up.
enum { kSpanBefore = 0, kSpanAfter = 1, kSpanWhole = 2 };
__device__ __forceinline__ uint32_t graph_span(const int64_t *vtx_off, uint32_t g, uint32_t x0,
                                               uint32_t vshift) {
    if (vtx_off[g] < (int64_t)x0) return kSpanBefore;
    return vtx_off[g + 1] > (int64_t)x0 + (1ll << vshift) ? kSpanAfter : kSpanWhole;
}

// batched counting over the union's oriented rows (batched.hip): row x is fcol[frow[x].x ..
// frow[x].y), ids of the union
struct BatchKernelArgs {
    const uint2 *frow;
    const uint32_t *fcol, *gid;
    const uint2 *items;       // heavy items (row, first entry); *n_items of them
    const uint32_t *n_items;
    const uint32_t *n;        // vertices (device)
    const int64_t *const *vtx_off_pp;  // the graphs' vertex offsets
    unsigned long long *wtotal;        // the waves' parts of graphs that span waves
    uint32_t *queue;
    unsigned long long *const *totals_pp;
    unsigned long long *const *tpv_pp;
    uint32_t kitem;       // entries per heavy item
    uint32_t light_max;   // rows with at most this many forward entries are light (<= 256)
    uint32_t wave_bits;   // heavy items use a bitmap below this id span (<= kWaveBits)
    uint32_t wave_list;   // ... else a sorted LDS list of at most this many entries
    uint32_t window;      // entries of light rows staged at a time (count_light_window)
};
// heavy items on heavy_wgs workgroups; light rows of up to ncap vertices, one wave per
// 2^vshift of them
hipError_t launch_count_u(const BatchKernelArgs &a, bool per_vertex, uint32_t heavy_wgs,
                          uint32_t ncap, uint32_t vshift, hipStream_t s);
// batched kernels: rows with at most count_light_max() forward entries are counted edge by
// edge, count_light_window(chunk, light_max) staged entries at a time
uint32_t count_light_max();
uint32_t count_light_chunk_max();
uint32_t count_light_window(uint32_t chunk, uint32_t light_max);

}  // namespace tc
