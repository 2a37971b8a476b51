// Device-wide exclusive scan and stable LSD radix sort of uint64 keys.
//
// The sort replaces the library sort of packed 64-bit edge keys in the preprocessing phase
// (Section 3.2, step 3, and the note on sorting edges as 64-bit integers): keys are ordered
// on a bit range [lo_bit, hi_bit) with digits of 8 or 9 bits (digit_bits), least significant
// digit first; a pass is an upsweep (per-tile digit histograms), an exclusive scan of the
// digit-major histogram table, and a stable scatter in which every wave ranks its own contiguous
// part of the tile with ballots, the tile is ordered by digit in LDS, and every digit's run is
// written out contiguously.  Up to kRawTiles tiles the scatter adds up the unscanned table itself,
// and a single tile needs no upsweep either.
//
// Single-sweep variant (large sorts that report errors through a status word): one upfront
// kernel counts the digits of every pass over all keys; each pass is then one kernel whose
// tiles take consecutive ids in launch order, publish their digit counts, and add up their
// predecessors' published counts (decoupled look-back) instead of reading a scanned table,
// which saves the upsweep's read of every key and the scan per pass.  A tile only waits on
// tiles that started before it and publish before they wait themselves, so the waits end;
// every wait is also bounded and reports TC_E_HIP if the bound is ever reached.
#include <type_traits>

#include "internal.h"

namespace tc {

// ======================================================================= fill

// Several arrays cleared by one launch: blockIdx.y picks the array (16-byte aligned), its blocks
// stride over it.
__global__ __launch_bounds__(256) void k_fill(const FillList f) {
    const Fill a = f.a[blockIdx.y];
    const uint64_t stride = (uint64_t)gridDim.x * 256, quads = a.words / 4;
    uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < a.words % 4) a.p[quads * 4 + i] = a.value;
    const uint4 v = make_uint4(a.value, a.value, a.value, a.value);
    for (; i < quads; i += stride) reinterpret_cast<uint4 *>(a.p)[i] = v;
}

hipError_t fill_all(const FillList &f, hipStream_t s) {
    uint64_t most = 0;
    for (int k = 0; k < f.count; ++k) most = f.a[k].words > most ? f.a[k].words : most;
    if (most == 0) return hipSuccess;
    const uint64_t blocks = (most / 4 + 256) / 256;
    hipLaunchKernelGGL(k_fill, dim3((uint32_t)(blocks < 8192 ? blocks : 8192), (uint32_t)f.count),
                       dim3(256), 0, s, f);
    return hipGetLastError();
}

hipError_t fill_u32(uint32_t *p, uint32_t value, uint64_t count, hipStream_t s) {
    FillList f;
    f.add(p, value, count);
    return fill_all(f, s);
}

// ======================================================================= scan

// A tile is 16384 elements for 1024 threads: four rows of 4096, four consecutive elements per
// thread and row (16-byte loads and stores, no transposition through LDS).  Up to one tile, one
// launch; beyond, two: the tile totals, then the scan, each workgroup adding up the totals
// before its own tile itself (at most 2^15 of them for 2^29 elements) instead of reading a
// scanned table.  The scans of the preprocessing are bound by their launches, not by memory:
// with 4096-element tiles and three to five launches each they took 260 of the 2150 us of a
// count at R-MAT scale 20 and 125 of 385 us at 100,003 edges.
constexpr int kScanThreads = 1024;
constexpr int kScanRows = 4;
constexpr int kScanWaves = kScanThreads / kWave;                // 16
constexpr uint32_t kScanRow = kScanThreads * 4;                 // 4096
constexpr uint32_t kScanTile = kScanRow * kScanRows;            // 16384
static_assert(kScanRows * kScanWaves == kWave, "one wave scans the row-wave totals");

// What a scan adds up: an array, or values formed from the arrays behind them, so that they need
// no launch and no array of their own.  at(y, i, N): elements i .. i + 3 of sequence y (0 from N on).
// (in 16-byte loads: with one 4-byte load per element a scan of 100,003 rows took 10 us instead
// of 3)
__device__ __forceinline__ uint4 load_four(const uint32_t *in, uint64_t i, uint64_t N) {
    if (i + 4 <= N) return *reinterpret_cast<const uint4 *>(in + i);
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (i < N) x.x = in[i];
    if (i + 1 < N) x.y = in[i + 1];
    if (i + 2 < N) x.z = in[i + 2];
    return x;
}
struct ScanArrays {  // sequence y: an array (16-byte aligned)
    const uint32_t *p[4];
    __device__ __forceinline__ uint4 at(uint32_t y, uint64_t i, uint64_t N) const {
        return load_four(p[y], i, N);
    }
};
struct ScanRows {  // row lengths from the rows' bounds (both 0 for an empty row)
    const uint32_t *rs, *re;
    __device__ __forceinline__ uint4 at(uint32_t, uint64_t i, uint64_t N) const {
        const uint4 a = load_four(rs, i, N), b = load_four(re, i, N);
        return make_uint4(b.x - a.x, b.y - a.y, b.z - a.z, b.w - a.w);
    }
};
// Room of every row's entries >= hbase in hcol: none for a row without such entries, else their
// number rounded up to a multiple of 8, plus `pad` zeros (the counting kernel's pieces, read
// from 8-aligned positions inside the row's part, never leave it).  row_ptr has N + 1 elements.
struct ScanHigh {
    const uint32_t *row_ptr, *hrow;
    uint32_t pad;
    __device__ __forceinline__ uint32_t room(uint32_t end, uint32_t h) const {
        return h != ~0u ? ((end - h + 7u) & ~7u) + pad : 0u;
    }
    __device__ __forceinline__ uint4 at(uint32_t, uint64_t i, uint64_t N) const {
        if (i >= N) return make_uint4(0u, 0u, 0u, 0u);
        const uint4 h = load_four(hrow, i, N), r = load_four(row_ptr, i, N + 1);
        uint4 x = make_uint4(room(r.y, h.x), 0u, 0u, 0u);
        if (i + 1 < N) x.y = room(r.z, h.y);
        if (i + 2 < N) x.z = room(r.w, h.z);
        if (i + 3 < N) x.w = room(row_ptr[i + 4], h.w);
        return x;
    }
};
struct ScanOut {
    uint32_t *p[4];
};

// sums[b] = total of tile b (of sequence y: after y * stride)
template <class In>
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(const In in, uint64_t N,
                                                            uint32_t *__restrict__ sums,
                                                            uint32_t stride) {
    __shared__ uint32_t s_wave[kScanWaves];
    const uint32_t t = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    uint32_t run = 0;
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        const uint4 x = in.at(blockIdx.y, base + r * kScanRow + t * 4, N);
        run += x.x + x.y + x.z + x.w;
    }
    run = wave_total(run);
    if (lane_id() == 0) s_wave[t / kWave] = run;
    __syncthreads();
    if (t < kWave) {
        const uint32_t total = wave_total(t < kScanWaves ? s_wave[t] : 0u);
        if (t == 0) sums[blockIdx.y * stride + blockIdx.x] = total;
    }
}

// out[i] = sum of the elements before i, for i < N + tail (the elements from N on are 0), of tile
// b, after the totals of the tiles before it (an input array may be its output: a workgroup
// reads its whole tile before it writes)
template <class In>
__global__ __launch_bounds__(kScanThreads) void k_scan_tile(const In in, const ScanOut outs,
                                                            uint64_t N, uint32_t tail,
                                                            const uint32_t *__restrict__ sums,
                                                            uint32_t stride) {
    __shared__ uint32_t s_part[kScanRows * kScanWaves], s_carry[kScanWaves];
    const uint32_t t = threadIdx.x, w = t / kWave, lane = lane_id();
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile, M = N + tail;
    uint32_t *out = outs.p[blockIdx.y];
    uint4 x[kScanRows];
    uint32_t incl[kScanRows];
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) x[r] = in.at(blockIdx.y, base + r * kScanRow + t * 4, N);
    uint32_t before = 0;
    for (uint32_t k = t; k < blockIdx.x; k += kScanThreads) before += sums[blockIdx.y * stride + k];
    before = wave_total(before);
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        incl[r] = wave_incl_scan(x[r].x + x[r].y + x[r].z + x[r].w);
        if (lane == kWave - 1) s_part[r * kScanWaves + w] = incl[r];
    }
    if (lane == 0) s_carry[w] = before;
    __syncthreads();
    // every wave scans the 64 (row, wave) totals in element order and adds up the carries
    const uint32_t part = s_part[lane];
    const uint32_t excl = wave_incl_scan(part) - part;
    const uint32_t carry = wave_total(lane < kScanWaves ? s_carry[lane] : 0u);
#pragma unroll
    for (int r = 0; r < kScanRows; ++r) {
        const uint64_t i = base + r * kScanRow + t * 4;
        const uint32_t off = (uint32_t)__builtin_amdgcn_readlane((int)excl, r * kScanWaves + w);
        uint4 y;
        y.x = carry + off + incl[r] - (x[r].x + x[r].y + x[r].z + x[r].w);
        y.y = y.x + x[r].x;
        y.z = y.y + x[r].y;
        y.w = y.z + x[r].z;
        if (i + 4 <= M) {
            *reinterpret_cast<uint4 *>(out + i) = y;
        } else {
            if (i < M) out[i] = y.x;
            if (i + 1 < M) out[i + 1] = y.y;
            if (i + 2 < M) out[i + 2] = y.z;
        }
    }
}

size_t scan_scratch_words(uint64_t N) {  // up to four sequences of N elements
    return (size_t)align_up(4 * ((N + kScanTile - 1) / kScanTile + 1), 64);
}

template <class In>
static hipError_t scan_any(const In &in, const ScanOut &out, uint32_t seqs, uint64_t N,
                           uint32_t tail, uint32_t *scratch, hipStream_t s) {
    if (N + tail == 0) return hipSuccess;
    const uint32_t nb = ceil_div(N + tail, kScanTile);
    if (nb > 1) {
        hipLaunchKernelGGL(k_scan_sums<In>, dim3(nb, seqs), dim3(kScanThreads), 0, s, in, N,
                           scratch, nb);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_scan_tile<In>, dim3(nb, seqs), dim3(kScanThreads), 0, s, in, out, N, tail,
                       scratch, nb);
    return hipGetLastError();
}

hipError_t scan_exclusive_u32(const uint32_t *in, uint32_t *out, uint64_t N, uint32_t *scratch,
                              hipStream_t s) {
    return scan_any(ScanArrays{{in, in, in, in}}, ScanOut{{out, out, out, out}}, 1, N, 0, scratch,
                    s);
}
hipError_t scan_four_u32(uint32_t *const in[4], uint32_t *const out[4], uint64_t N,
                         uint32_t *scratch, hipStream_t s) {
    return scan_any(ScanArrays{{in[0], in[1], in[2], in[3]}},
                    ScanOut{{out[0], out[1], out[2], out[3]}}, 4, N, 0, scratch, s);
}
hipError_t scan_row_bounds(const uint32_t *rs, const uint32_t *re, uint64_t rows, uint32_t *out,
                           uint32_t *scratch, hipStream_t s) {
    return scan_any(ScanRows{rs, re}, ScanOut{{out, out, out, out}}, 1, rows, 1, scratch, s);
}
hipError_t scan_high_rows(const uint32_t *row_ptr, const uint32_t *hrow, uint64_t rows,
                          uint32_t pad, uint32_t *out, uint32_t *scratch, hipStream_t s) {
    return scan_any(ScanHigh{row_ptr, hrow, pad}, ScanOut{{out, out, out, out}}, 1, rows, 1,
                    scratch, s);
}

// ======================================================================= radix sort

// A tile is 8192 keys for 512 threads; wave w owns the contiguous keys [1024 w, 1024 (w + 1))
// of the tile as 16 rows of 64, so that a wave ranks its keys with counters of its own and
// the tile needs no barrier per row: the stable order of the tile is wave by wave, row by
// row, lane by lane.
constexpr int kSortThreads = 512;
constexpr int kSortItems = 16;
constexpr int kSortWaves = kSortThreads / kWave;     // 8
constexpr int kSortTile = kSortThreads * kSortItems;  // 8192 keys per tile

// Lanes holding the same kBits-bit digit as the calling lane: returns the mask of such (valid)
// lanes.  Per bit: m = all ones where the lane's bit is set, the ballot of that bit, and
// peers &= ~(ballot ^ m) on both halves.
template <int kBits>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid) {
    const uint64_t v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
        const uint32_t m = (uint32_t)((int32_t)(d << (31 - b)) >> 31);
        const uint64_t bb = __ballot(m != 0u);
        lo &= ~((uint32_t)bb ^ m);
        hi &= ~((uint32_t)(bb >> 32) ^ m);
    }
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t tile_key_index(uint64_t base, uint32_t w, int r) {
    return base + (uint64_t)w * (kSortItems * kWave) + (uint64_t)r * kWave + lane_id();
}

// Where a pass reads its keys: 64-bit keys, or (for the first pass of a sort of keys
// (value << 32) | position) 32-bit values whose key is formed with the value's own index, so
// that the producer writes and the first pass reads 4 bytes per key instead of 8.
// keep(key): whether the pass takes the key (the others are dropped, and the output holds
// only the kept keys, in order).
struct Keys64 {  // (read once per pass, with a non-temporal hint: no reuse within a pass)
    const uint64_t *p;
    __device__ __forceinline__ uint64_t operator()(uint64_t i) const {
        return __builtin_nontemporal_load(p + i);
    }
    __device__ __forceinline__ bool keep(uint64_t) const { return true; }
};
struct KeysHiIndex {  // drops the keys whose value is `drop`
    const uint32_t *p;
    uint32_t drop;
    __device__ __forceinline__ uint64_t operator()(uint64_t i) const {
        return ((uint64_t)__builtin_nontemporal_load(p + i) << 32) | (uint32_t)i;
    }
    __device__ __forceinline__ bool keep(uint64_t key) const {
        return (uint32_t)(key >> 32) != drop;
    }
};

// the vertex order's first pass: vertex i's key (degree << b) | i, formed from the degrees
struct KeysDegree {
    const uint32_t *deg;
    int b;
    __device__ __forceinline__ uint64_t operator()(uint64_t i) const {
        const uint64_t lim = (1ull << b) - 1, d = deg[i];
        return ((d < lim ? d : lim) << b) | i;  // (above lim only for invalid input)
    }
    __device__ __forceinline__ bool keep(uint64_t) const { return true; }
};

// Where a pass writes its keys: 64-bit keys, or split for the last pass of the in-edge list
// sort into the list id (high half) and the list entry cbeg = position + 1 (low half + 1).
struct Out64 {
    uint64_t *p;
    __device__ __forceinline__ void operator()(uint64_t pos, uint64_t key) const { p[pos] = key; }
};
// ... or unzipped, for the last pass of the edge sort: target (low b bits) and source.
struct OutColSrc {
    uint32_t *col, *src;
    uint64_t tmask;
    int b;
    __device__ __forceinline__ void operator()(uint64_t pos, uint64_t key) const {
        col[pos] = (uint32_t)(key & tmask);
        src[pos] = (uint32_t)(key >> b);
    }
};
// ... or, for the last pass of the vertex order: perm[r] = the vertex (low b bits) of the key
// at position r, rank[vertex] = r.
struct OutPermRank {
    uint32_t *perm, *rank;
    uint64_t mask;
    __device__ __forceinline__ void operator()(uint64_t pos, uint64_t key) const {
        const uint32_t x = (uint32_t)(key & mask);
        perm[pos] = x;
        rank[x] = (uint32_t)pos;
    }
};
struct OutListBeg {
    uint32_t *list, *beg;
    __device__ __forceinline__ void operator()(uint64_t pos, uint64_t key) const {
        list[pos] = (uint32_t)(key >> 32);
        beg[pos] = (uint32_t)key + 1u;
    }
};

// Loads the calling wave's 16 rows of the tile (all loads in flight before any use) and
// returns the lane's mask of rows whose key takes part (below count, and kept);
// kFull: the whole tile lies below count.
template <bool kFull, class Src>
__device__ __forceinline__ uint32_t load_tile_keys(const Src in, uint32_t count, uint64_t base,
                                                   uint32_t w, uint64_t (&keys)[kSortItems]) {
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint64_t idx = tile_key_index(base, w, r);
        keys[r] = (kFull || idx < count) ? in(idx) : 0ull;
    }
    uint32_t vmask = 0;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint64_t idx = tile_key_index(base, w, r);
        if ((kFull || idx < count) && in.keep(keys[r])) vmask |= 1u << r;
    }
    return vmask;
}

// Digits of 8 bits, or 9 where that saves a pass (digit_bits).  With counters of 16 bits the
// state of a tile with 512 digits (76 KB; a tile has 8192 keys) leaves room for two workgroups
// per CU as with 256.
template <int kBits>
using TileCount = std::conditional_t<kBits == 8, uint32_t, uint16_t>;

// Per-wave digit counts of the wave's rows into cnt[] (the wave's own row of counters,
// zero on entry), and each key's rank among the wave's earlier keys of the same digit.
template <int kBits>
__device__ __forceinline__ void wave_rank_rows(const uint64_t (&keys)[kSortItems], uint32_t vmask,
                                               int shift, uint32_t mask, TileCount<kBits> *cnt,
                                               uint32_t (&ranks)[kSortItems]) {
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const bool valid = (vmask >> r) & 1u;
        const uint32_t d = (uint32_t)(keys[r] >> shift) & mask;
        const uint64_t peers = match_digit<kBits>(d, valid);
        const uint32_t below = lanes_below(peers);
        const uint32_t prev = valid ? cnt[d] : 0u;
        ranks[r] = prev + below;
        if (valid && below == 0) cnt[d] = (TileCount<kBits>)(prev + (uint32_t)__popcll(peers));
        wave_lds_sync();  // this row's counter updates before the next row's reads
    }
}

// Shared state of one tile's stable placement in digit order.
template <int kBits>
struct SortTileLds {
    static constexpr uint32_t kDigits = 1u << kBits;
    static_assert(kDigits <= kSortThreads, "one thread per digit");
    uint64_t stage[kSortTile];
    // per-wave digit counts, then per-wave digit offsets
    TileCount<kBits> wcnt[kSortWaves][kDigits];
    uint32_t loc[kDigits];           // tile-local start of each digit
    uint32_t glob[kDigits];          // global start minus local start of each digit
    uint32_t dsum[kDigits / kWave];  // per-wave sums of the digit scan
    uint32_t gsum[4];                // the same for the global digit counts (single sweep)
    uint32_t gwave[kSortWaves];      // per-wave sums of the global counts (few tiles)
    uint32_t total;                  // keys of the tile that take part
};

// Block part of the placement (all threads, after the waves' counts are in wcnt): turns wcnt
// into per-wave digit offsets, fills loc, and returns the tile's count of digit t.
template <int kBits>
__device__ __forceinline__ uint32_t tile_digit_offsets(SortTileLds<kBits> &L) {
    constexpr uint32_t kDigits = 1u << kBits;
    const uint32_t t = threadIdx.x;
    __syncthreads();
    uint32_t c = 0;
    if (t < kDigits) {
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) {
            const uint32_t x = L.wcnt[k][t];
            L.wcnt[k][t] = (TileCount<kBits>)c;
            c += x;
        }
    }
    const uint32_t incl = wave_incl_scan(t < kDigits ? c : 0u);
    if (t < kDigits && lane_id() == kWave - 1) L.dsum[t / kWave] = incl;
    __syncthreads();
    if (t < kDigits) {
        uint32_t before = 0;
        for (uint32_t k = 0; k < t / kWave; ++k) before += L.dsum[k];
        L.loc[t] = before + incl - c;
        if (t == kDigits - 1) L.total = before + incl;
    }
    return c;
}

// Places the wave's keys in L.stage (after tile_digit_offsets and a barrier).
template <int kBits>
__device__ __forceinline__ void stage_keys(SortTileLds<kBits> &L, const uint64_t (&keys)[kSortItems],
                                           const uint32_t (&ranks)[kSortItems], uint32_t vmask,
                                           uint32_t w, int shift, uint32_t mask) {
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        if ((vmask >> r) & 1u) {
            const uint32_t d = (uint32_t)(keys[r] >> shift) & mask;
            L.stage[L.loc[d] + L.wcnt[w][d] + ranks[r]] = keys[r];
        }
    }
}

// Writes the staged tile (L.total keys): consecutive threads write consecutive positions of
// one digit's run (L.glob[d] + j is the output position of staged key j of digit d).
template <int kBits, class Dst>
__device__ __forceinline__ void write_staged(const SortTileLds<kBits> &L, const Dst out, uint32_t count,
                                             int shift, uint32_t mask, int32_t *status) {
    const uint32_t ntile = L.total;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const uint32_t j = (uint32_t)i * kSortThreads + threadIdx.x;
        if (j < ntile) {
            const uint64_t key = L.stage[j];
            const uint32_t d = (uint32_t)(key >> shift) & mask;
            const uint32_t pos = L.glob[d] + j;
            if (!status) {
                out(pos, key);
            } else if (pos < count) {  // holds whenever the prefixes are right
                out(pos, key);
            } else {
                set_status(status, TC_E_HIP);
            }
        }
    }
}

template <int kBits, bool kFull, class Src>
__device__ __forceinline__ void hist_tile(const Src in, uint32_t count, int shift,
                                          uint32_t mask, uint32_t *__restrict__ hist,
                                          uint32_t tiles, uint32_t tile,
                                          uint32_t (&h)[kSortWaves][1 << kBits]) {
    const uint32_t t = threadIdx.x, w = t / kWave;
    const uint64_t base = (uint64_t)tile * kSortTile;
    uint64_t keys[kSortItems];
    const uint32_t vmask = load_tile_keys<kFull>(in, count, base, w, keys);
    for (uint32_t k = lane_id(); k < 1u << kBits; k += kWave) h[w][k] = 0;
    wave_lds_sync();
    // counts only (no ranks): the keys of a row that share the first lane's digit are added
    // with one LDS atomic, the others one atomic each, into the wave's own counters (skewed
    // keys -- hub ranks, long runs of equal digits after the first pass -- would otherwise
    // serialise many atomics on one counter)
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const bool valid = (vmask >> r) & 1u;
        const uint32_t d = (uint32_t)(keys[r] >> shift) & mask;
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
        const uint64_t same = __ballot(valid && d == d0);
        if (lane_id() == 0 && same) atomicAdd(&h[w][d0], (uint32_t)__popcll(same));
        if (valid && d != d0) atomicAdd(&h[w][d], 1u);
    }
    __syncthreads();
    if (t < 1u << kBits) {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) sum += h[k][t];
        hist[(uint64_t)t * tiles + tile] = sum;
    }
}

// dcount (nullable): the number of keys, read from the device (a bound set by an earlier pass
// that dropped keys; count is then the capacity the grid was sized for)
template <int kBits, class Src>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const Src in, uint32_t count,
                                                             const uint32_t *__restrict__ dcount,
                                                             int shift, uint32_t nbits,
                                                             uint32_t *__restrict__ hist,
                                                             uint32_t tiles,
                                                             const int32_t *__restrict__ status) {
    if (status && *status) return;
    if (dcount) count = min(count, *dcount);
    __shared__ uint32_t h[kSortWaves][1 << kBits];
    const uint32_t tile = xcd_tile(blockIdx.x, tiles);
    const uint32_t mask = (1u << nbits) - 1u;
    if ((uint64_t)(tile + 1) * kSortTile <= count)
        hist_tile<kBits, true>(in, count, shift, mask, hist, tiles, tile, h);
    else
        hist_tile<kBits, false>(in, count, shift, mask, hist, tiles, tile, h);
}

// How a scatter finds where its tile's digit runs start.  Few tiles (at most kRawTiles): from the
// per-tile counts themselves, the digits' rows of the table added up by the waves, which saves
// the scan's launches (a sort of 100,003 keys is bound by its launches, 4 to 10 us each: a whole
// count of such a graph went from 384 to 309 us with this and the two-launch scan); a single
// tile needs no table at all.  More tiles: from the scanned table (every workgroup would read
// the whole table otherwise, 128 KB at 128 tiles).
constexpr uint32_t kRawTiles = 128;
// Up to kColumnTiles tiles, one thread adds up a digit's row (its loads are a row apart, so their
// lines grow with the tiles); more, a wave adds up 32 digits' rows at a time, one scan each, 64 for
// a wave with 512 digits whatever the tiles.  A sort on 63 bits, us, by waves and by threads: 20,000
// keys (3 tiles) 165 and 109, 131,072 (16) 169 and 136, 262,144 (32) 172 and 164, 400,000 (49) 177
// and 195.  (With the scan's launches, as for many tiles, it takes 137 for 20,000.)
constexpr uint32_t kColumnTiles = 32;

// Global minus local start of every digit into L.glob (all threads; loc filled).
// (kFew: at most kRawTiles tiles; an instance of its own, since its registers would halve the
// occupancy of the other)
template <int kBits, bool kFew>
__device__ __forceinline__ void tile_digit_starts(SortTileLds<kBits> &L,
                                                  const uint32_t *__restrict__ table,
                                                  uint32_t tiles, uint32_t tile) {
    constexpr uint32_t kDigits = 1u << kBits;
    const uint32_t t = threadIdx.x;
    if constexpr (!kFew) {
        if (t < kDigits) L.glob[t] = table[(uint64_t)t * tiles + tile] - L.loc[t];
    } else if (tiles == 1) {
        if (t < kDigits) L.glob[t] = 0;
    } else if (tiles <= kColumnTiles) {
        constexpr uint32_t kStep = 8;
        const uint32_t w = t / kWave;
        uint32_t sum = 0, below = 0;
        for (uint32_t k0 = 0; t < kDigits && k0 < tiles; k0 += kStep) {
            uint32_t x[kStep];
#pragma unroll
            for (uint32_t k = 0; k < kStep; ++k)
                x[k] = k0 + k < tiles ? table[t * tiles + k0 + k] : 0u;
#pragma unroll
            for (uint32_t k = 0; k < kStep; ++k) {
                sum += x[k];
                below += k0 + k < tile ? x[k] : 0u;
            }
        }
        const uint32_t incl = wave_incl_scan(sum);
        if (lane_id() == kWave - 1) L.gwave[w] = incl;
        __syncthreads();
        uint32_t before = 0;
        for (uint32_t k = 0; k < w; ++k) before += L.gwave[k];
        if (t < kDigits) L.glob[t] = before + incl - sum + below - L.loc[t];
    } else {
        // a wave sums its digits' rows, 32 at a time, lanes along the tiles; lane i keeps its
        // digit i's sums
        constexpr uint32_t kMine = kDigits / kSortWaves, kStep = 32;
        const uint32_t w = t / kWave, lane = lane_id();
        uint32_t sum = 0, below = 0;
        for (uint32_t i0 = 0; i0 < kMine; i0 += kStep) {
            for (uint32_t k0 = 0; k0 < tiles; k0 += kWave) {
                const uint32_t k = k0 + lane;
                uint32_t x[kStep];  // (all loads in flight together)
#pragma unroll
                for (uint32_t i = 0; i < kStep; ++i)
                    x[i] = k < tiles ? table[(w * kMine + i0 + i) * tiles + k] : 0u;
#pragma unroll
                for (uint32_t i = 0; i < kStep; ++i) {
                    const uint32_t in = wave_incl_scan(x[i]);
                    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)in, kWave - 1);
                    // the tiles before this one: all of the 64, or those up to its own lane
                    const uint32_t part =
                        tile >= k0 + kWave ? all
                        : tile > k0
                            ? (uint32_t)__builtin_amdgcn_readlane((int)in, (int)(tile - 1 - k0))
                            : 0u;
                    if (lane == i0 + i) {
                        sum += all;
                        below += part;
                    }
                }
            }
        }
        const uint32_t incl = wave_incl_scan(sum);  // (lanes from kMine on hold 0)
        if (lane == kWave - 1) L.gwave[w] = incl;
        __syncthreads();
        uint32_t before = 0;
        for (uint32_t k = 0; k < w; ++k) before += L.gwave[k];
        if (lane < kMine) {
            const uint32_t d = w * kMine + lane;
            L.glob[d] = before + incl - sum + below - L.loc[d];
        }
    }
}

// Stable scatter of one tile: the keys are ranked and placed in LDS in digit order (a
// tile-local counting sort), then written out digit run by digit run.
//   table: digit-major per-tile digit counts, scanned when there are more than kRawTiles tiles
//   total: nullable, receives the number of keys of all tiles
template <int kBits, bool kFull, bool kFew, class Src, class Dst>
__device__ __forceinline__ void scatter_tile(const Src in, const Dst out, uint32_t count,
                                             int shift, uint32_t mask,
                                             const uint32_t *__restrict__ table, uint32_t tiles,
                                             uint32_t tile, uint32_t *__restrict__ total,
                                             SortTileLds<kBits> &L) {
    const uint32_t t = threadIdx.x, w = t / kWave;
    const uint64_t base = (uint64_t)tile * kSortTile;
    uint64_t keys[kSortItems];
    const uint32_t vmask = load_tile_keys<kFull>(in, count, base, w, keys);
    for (uint32_t k = lane_id(); k < 1u << kBits; k += kWave) L.wcnt[w][k] = 0;
    wave_lds_sync();
    uint32_t ranks[kSortItems];
    wave_rank_rows<kBits>(keys, vmask, shift, mask, L.wcnt[w], ranks);
    const uint32_t c = tile_digit_offsets(L);
    __syncthreads();
    tile_digit_starts<kBits, kFew>(L, table, tiles, tile);
    __syncthreads();
    // the last tile's last run ends at the number of keys
    constexpr uint32_t kLast = (1u << kBits) - 1u;
    if (total && tile == tiles - 1 && t == kLast) *total = L.glob[kLast] + L.loc[kLast] + c;
    stage_keys(L, keys, ranks, vmask, w, shift, mask);
    __syncthreads();
    write_staged(L, out, count, shift, mask, nullptr);
}

template <int kBits, bool kFew, class Src, class Dst>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const Src in, const Dst out, uint32_t count, const uint32_t *__restrict__ dcount, int shift,
    uint32_t nbits, const uint32_t *__restrict__ table, uint32_t tiles,
    uint32_t *__restrict__ total, const int32_t *__restrict__ status) {
    if (status && *status) return;
    if (dcount) count = min(count, *dcount);
    __shared__ SortTileLds<kBits> L;
    const uint32_t tile = xcd_tile(blockIdx.x, tiles);
    if ((uint64_t)tile * kSortTile >= count) return;  // past the keys (a device count)
    const uint32_t mask = (1u << nbits) - 1u;
    if ((uint64_t)(tile + 1) * kSortTile <= count)
        scatter_tile<kBits, true, kFew>(in, out, count, shift, mask, table, tiles, tile, total, L);
    else
        scatter_tile<kBits, false, kFew>(in, out, count, shift, mask, table, tiles, tile, total, L);
}

// ---------------------------------------------------------------- single-sweep variant

constexpr uint32_t kLbAgg = 1u << 30;       // published: this tile's own count
constexpr uint32_t kLbIncl = 2u << 30;      // published: inclusive prefix up to this tile
constexpr uint32_t kLbValue = (1u << 30) - 1u;
constexpr uint32_t kLbMaxPolls = 1u << 20;  // bound on the polls of one look-back
constexpr uint32_t kLbWindow = 16;          // predecessors' flags read per round trip
constexpr int kMaxPasses = 8;

// digit counts of every pass over all keys: ghist[p * 256 + d]
__global__ __launch_bounds__(256) void k_radix_digits(
    const uint64_t *__restrict__ in, uint32_t count, int lo_bit, int passes, int hi_bit,
    uint32_t *__restrict__ ghist, const int32_t *__restrict__ status) {
    if (*status) return;
    __shared__ uint32_t h[kMaxPasses][256];
    const uint32_t t = threadIdx.x;
    for (int p = 0; p < kMaxPasses; ++p) h[p][t] = 0;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + t; i < count; i += stride) {
        const uint64_t k = in[i];
        for (int p = 0; p < passes; ++p) {
            const int sh = lo_bit + 8 * p;
            const uint32_t nb = (hi_bit - sh) < 8 ? (uint32_t)(hi_bit - sh) : 8u;
            atomicAdd(&h[p][(uint32_t)(k >> sh) & ((1u << nb) - 1u)], 1u);
        }
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p)
        if (h[p][t]) atomicAdd(&ghist[p * 256 + t], h[p][t]);
}

// One pass: tile ids in launch order; flags[tile * 256 + d] = kLbAgg | count, then
// kLbIncl | inclusive prefix, of digit d.
template <bool kFull>
__device__ __forceinline__ void onesweep_tile(const uint64_t *__restrict__ in,
                                              uint64_t *__restrict__ out, uint32_t count,
                                              int shift, uint32_t mask,
                                              const uint32_t *__restrict__ ghist,
                                              uint32_t *__restrict__ flags, uint32_t tile,
                                              int32_t *__restrict__ status, SortTileLds<8> &L) {
    const uint32_t t = threadIdx.x, w = t / kWave;
    const uint64_t base = (uint64_t)tile * kSortTile;
    uint64_t keys[kSortItems];
    const uint32_t vmask = load_tile_keys<kFull>(Keys64{in}, count, base, w, keys);
    for (uint32_t k = lane_id(); k < 256; k += kWave) L.wcnt[w][k] = 0;
    wave_lds_sync();
    uint32_t ranks[kSortItems];
    wave_rank_rows<8>(keys, vmask, shift, mask, L.wcnt[w], ranks);
    const uint32_t c = tile_digit_offsets(L);
    if (t < 256)
        __hip_atomic_store(&flags[(uint64_t)tile * 256 + t], (tile == 0 ? kLbIncl : kLbAgg) | c,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the global start of every digit
    const uint32_t gc = t < 256 ? ghist[t] : 0u;
    const uint32_t gincl = wave_incl_scan(gc);
    if (t < 256 && lane_id() == kWave - 1) L.gsum[w] = gincl;
    __syncthreads();
    stage_keys(L, keys, ranks, vmask, w, shift, mask);
    if (t < 256) {
        uint32_t gbefore = 0;
        for (uint32_t k = 0; k < w; ++k) gbefore += L.gsum[k];
        const uint32_t gstart = gbefore + gincl - gc;
        // look-back: keys of digit t in the tiles before this one.  The flags of kLbWindow
        // predecessors are read together (one memory round trip instead of one per tile) and
        // taken nearest first until an inclusive prefix; an unpublished flag is waited for
        uint32_t excl = 0;
        if (tile > 0) {
            uint32_t j = tile - 1, polls = 0;
            bool done = false;
            while (!done) {
                uint32_t f[kLbWindow];
#pragma unroll
                for (uint32_t i = 0; i < kLbWindow; ++i)
                    f[i] = i <= j ? __hip_atomic_load(&flags[(uint64_t)(j - i) * 256 + t],
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                  : kLbIncl;  // never reached: tile 0 is inclusive
                uint32_t taken = 0;
                bool wait = false;
#pragma unroll
                for (uint32_t i = 0; i < kLbWindow; ++i) {
                    if (done || wait) continue;
                    if ((f[i] & ~kLbValue) == 0) {
                        wait = true;
                        continue;
                    }
                    excl += f[i] & kLbValue;
                    ++taken;
                    if (f[i] & kLbIncl) done = true;
                }
                if (done) break;
                j -= taken;  // tile 0 publishes an inclusive prefix, so j never passes it
                if (wait) {
                    if (++polls >= kLbMaxPolls) {
                        set_status(status, TC_E_HIP);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __hip_atomic_store(&flags[(uint64_t)tile * 256 + t], kLbIncl | (excl + c),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        L.glob[t] = gstart + excl - L.loc[t];
    }
    __syncthreads();
    write_staged(L, Out64{out}, count, shift, mask, status);
}

__global__ __launch_bounds__(kSortThreads) void k_radix_onesweep(
    const uint64_t *__restrict__ in, uint64_t *__restrict__ out, uint32_t count, int shift,
    uint32_t nbits, const uint32_t *__restrict__ ghist, uint32_t *__restrict__ flags,
    uint32_t *__restrict__ tile_counter, int32_t *__restrict__ status) {
    __shared__ SortTileLds<8> L;
    __shared__ uint32_t s_tile;
    __shared__ int s_stop;
    if (threadIdx.x == 0) {
        s_tile = atomicAdd(tile_counter, 1u);
        s_stop = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    }
    __syncthreads();
    // after an error (earlier kernels, or a look-back bound reached in this one) tiles stop
    // before publishing; their successors' bounded waits end too
    if (s_stop) return;
    const uint32_t tile = s_tile;
    const uint32_t mask = (1u << nbits) - 1u;
    if ((uint64_t)(tile + 1) * kSortTile <= count)
        onesweep_tile<true>(in, out, count, shift, mask, ghist, flags, tile, status, L);
    else
        onesweep_tile<false>(in, out, count, shift, mask, ghist, flags, tile, status, L);
}

size_t sort_scratch_bytes(uint64_t count) {
    uint64_t tiles = (count + kSortTile - 1) / kSortTile;
    if (tiles == 0) tiles = 1;
    uint64_t hist = 256 * tiles;
    return 2 * align_up(hist * 4, 256) + align_up(scan_scratch_words(hist) * 4, 256);
}

// Bits per digit of the passes over a key of `bits` bits: 9 where that takes fewer passes than 8
// (9, 17, 18, 25 to 27, 33 to 36, 41 to 45, 49 to 54, 57 to 63 bits), and 8 elsewhere: a pass with 512 digits has a ninth
// ballot per key, twice the table and half the run length.  Preprocessing with digits of 8 and
// of 9 bits, us: 200,003 vertices and 3,000,001 edges 458 and 400, 262,144 and 20 million 1474
// and 1386, 2^25 and 100 million 11,840 and 11,080, 2^26 and 120 million 16,250 and 15,320.
// (Digits of 10 bits would need twice the scratch, and LDS for one workgroup per CU.)
static int digit_bits(int bits) { return (bits + 8) / 9 < (bits + 7) / 8 ? 9 : 8; }

template <int kBits, class Src, class Dst>
static hipError_t radix_pass_bits(const Src in, const Dst dst, uint32_t count, int shift,
                                  uint32_t nbits, void *scratch, int32_t *status, hipStream_t s,
                                  const uint32_t *dcount, uint32_t *total) {
    const uint32_t tiles = ceil_div(count, kSortTile);
    // scratch: two tables of 256 digits, or one of 512 that is scanned in place
    const size_t table_bytes = align_up(1024ull * tiles, 256);
    uint32_t *hist = (uint32_t *)scratch;
    uint32_t *offs = kBits == 8 ? (uint32_t *)((char *)scratch + table_bytes) : hist;
    uint32_t *scan_scratch = (uint32_t *)((char *)scratch + 2 * table_bytes);
    hipError_t e;
    if (tiles > 1) {
        hipLaunchKernelGGL((k_radix_hist<kBits, Src>), dim3(tiles), dim3(kSortThreads), 0, s, in,
                           count, dcount, shift, nbits, hist, tiles, status);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (tiles > kRawTiles) {
        e = scan_exclusive_u32(hist, offs, (uint64_t)tiles << kBits, scan_scratch, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_radix_scatter<kBits, false, Src, Dst>), dim3(tiles),
                           dim3(kSortThreads), 0, s, in, dst, count, dcount, shift, nbits, offs,
                           tiles, total, status);
    } else {
        hipLaunchKernelGGL((k_radix_scatter<kBits, true, Src, Dst>), dim3(tiles),
                           dim3(kSortThreads), 0, s, in, dst, count, dcount, shift, nbits, hist,
                           tiles, total, status);
    }
    return hipGetLastError();
}

// One stable two-kernel pass on the digit of up to `digit` bits at `shift` (below hi_bit) from
// the keys `in` yields to dst.  dcount (nullable): the number of keys on the device (count: the
// capacity); total (nullable): receives the number of keys written (the kept ones).
template <class Src, class Dst>
static hipError_t radix_pass(const Src in, const Dst dst, uint32_t count, int digit, int shift,
                             int hi_bit, void *scratch, int32_t *status, hipStream_t s,
                             const uint32_t *dcount = nullptr, uint32_t *total = nullptr) {
    const uint32_t nbits = (uint32_t)((hi_bit - shift) < digit ? (hi_bit - shift) : digit);
    return digit == 9 ? radix_pass_bits<9>(in, dst, count, shift, nbits, scratch, status, s,
                                           dcount, total)
                      : radix_pass_bits<8>(in, dst, count, shift, nbits, scratch, status, s,
                                           dcount, total);
}

// sort_u64 with digits of `digit` bits
static hipError_t sort_passes(uint64_t *keys, uint64_t *tmp, uint32_t count, int lo_bit,
                              int hi_bit, int digit, void *scratch, int32_t *status,
                              hipStream_t s, uint64_t **result, bool onesweep) {
    *result = keys;
    if (count <= 1 || hi_bit <= lo_bit) return hipSuccess;
    uint32_t tiles = ceil_div(count, kSortTile);
    uint64_t hist_n = 256ull * tiles;
    uint32_t *hist = (uint32_t *)scratch;
    uint32_t *offs = (uint32_t *)((char *)scratch + align_up(hist_n * 4, 256));
    uint64_t *src = keys, *dst = tmp;
    const int passes = (hi_bit - lo_bit + 7) / 8;
    if (status && onesweep && count >= (1u << 20) && count <= kLbValue &&
        hist_n >= (uint64_t)kMaxPasses * 256 + kMaxPasses) {
        // flags: the first table; digit counts and tile counters: the second
        uint32_t *flags = hist, *ghist = offs, *counters = offs + kMaxPasses * 256;
        hipError_t e = fill_u32(ghist, 0u, kMaxPasses * 256 + kMaxPasses, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_radix_digits, dim3(2048), dim3(256), 0, s, keys, count,
                           lo_bit, passes, hi_bit, ghist, status);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        for (int p = 0; p < passes; ++p) {
            const int shift = lo_bit + 8 * p;
            const uint32_t nbits = (uint32_t)((hi_bit - shift) < 8 ? (hi_bit - shift) : 8);
            if ((e = fill_u32(flags, 0u, hist_n, s)) != hipSuccess) return e;
            hipLaunchKernelGGL(k_radix_onesweep, dim3(tiles), dim3(kSortThreads), 0, s, src, dst,
                               count, shift, nbits, ghist + p * 256, flags, counters + p,
                               status);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            uint64_t *x = src;
            src = dst;
            dst = x;
        }
        *result = src;
        return hipSuccess;
    }
    for (int shift = lo_bit; shift < hi_bit; shift += digit) {
        hipError_t e =
            radix_pass(Keys64{src}, Out64{dst}, count, digit, shift, hi_bit, scratch, status, s);
        if (e != hipSuccess) return e;
        uint64_t *x = src;
        src = dst;
        dst = x;
    }
    *result = src;
    return hipSuccess;
}

hipError_t sort_u64(uint64_t *keys, uint64_t *tmp, uint32_t count, int lo_bit, int hi_bit,
                    void *scratch, int32_t *status, hipStream_t s, uint64_t **result,
                    bool onesweep) {
    return sort_passes(keys, tmp, count, lo_bit, hi_bit, digit_bits(hi_bit - lo_bit), scratch,
                       status, s, result, onesweep);
}

hipError_t sort_unzip(uint64_t *keys, uint64_t *tmp, uint32_t count, int lo_bit, int hi_bit,
                      int b, uint32_t *col, uint32_t *src, void *scratch, int32_t *status,
                      hipStream_t s, bool onesweep) {
    if (count == 0) return hipSuccess;
    // (a single sweep has digits of 8 bits)
    const int digit = onesweep ? 8 : digit_bits(hi_bit - lo_bit);
    const int passes = hi_bit > lo_bit ? (hi_bit - lo_bit + digit - 1) / digit : 1;
    const int last = hi_bit > lo_bit ? lo_bit + digit * (passes - 1) : hi_bit;
    uint64_t *mid = keys;
    hipError_t e = sort_passes(keys, tmp, count, lo_bit, last, digit, scratch, status, s, &mid,
                               onesweep);
    if (e != hipSuccess) return e;
    return radix_pass(Keys64{mid}, OutColSrc{col, src, (1ull << b) - 1, b}, count, digit, last,
                      hi_bit, scratch, status, s);
}

hipError_t sort_ranks(const uint32_t *deg, uint64_t *keys, uint64_t *tmp, uint32_t n, int b,
                      uint32_t *perm, uint32_t *rank, void *scratch, int32_t *status,
                      hipStream_t s) {
    if (n == 0) return hipSuccess;
    const KeysDegree first{deg, b};
    const OutPermRank last{perm, rank, (1ull << b) - 1};
    const int digit = digit_bits(b);
    if (b <= digit) return radix_pass(first, last, n, digit, b, 2 * b, scratch, status, s);
    hipError_t e = radix_pass(first, Out64{keys}, n, digit, b, 2 * b, scratch, status, s);
    uint64_t *src = keys, *dst = tmp;
    int shift = b + digit;
    for (; e == hipSuccess && shift + digit < 2 * b; shift += digit) {
        e = radix_pass(Keys64{src}, Out64{dst}, n, digit, shift, 2 * b, scratch, status, s);
        uint64_t *x = src;
        src = dst;
        dst = x;
    }
    if (e != hipSuccess) return e;
    return radix_pass(Keys64{src}, last, n, digit, shift, 2 * b, scratch, status, s);
}

hipError_t sort_lists(const uint32_t *cid, uint32_t drop, uint32_t count, int bits,
                      uint64_t *a, uint64_t *b, uint32_t *cbeg, uint32_t *kept, void *scratch,
                      int32_t *status, hipStream_t s, uint32_t **list) {
    *list = (uint32_t *)a;
    if (count == 0) return fill_u32(kept, 0u, 1, s);
    const int hi_bit = 32 + (bits > 0 ? bits : 0);
    const int digit = digit_bits(bits);
    const int passes = bits > 0 ? (bits + digit - 1) / digit : 1;
    const KeysHiIndex first{cid, drop};
    if (passes == 1)  // one pass from the ids to the split output
        return radix_pass(first, OutListBeg{*list, cbeg}, count, digit, 32, hi_bit, scratch, status, s,
                          nullptr, kept);
    hipError_t e =
        radix_pass(first, Out64{a}, count, digit, 32, hi_bit, scratch, status, s, nullptr, kept);
    if (e != hipSuccess) return e;
    uint64_t *src = a, *dst = b;
    for (int p = 1; p < passes - 1; ++p) {  // the middle passes, on the kept keys
        e = radix_pass(Keys64{src}, Out64{dst}, count, digit, 32 + digit * p, hi_bit, scratch,
                       status, s, kept);
        if (e != hipSuccess) return e;
        uint64_t *x = src;
        src = dst;
        dst = x;
    }
    *list = (uint32_t *)dst;  // the buffer the last pass does not read
    return radix_pass(Keys64{src}, OutListBeg{*list, cbeg}, count, digit,
                      32 + digit * (passes - 1), hi_bit, scratch, status, s, kept);
}

}  // namespace tc
