// Counting phase (Section 2.2 and Section 3.3): the sum over oriented edges u -> v of
// |N+(u) n N+(v)|.
//
// Vertices are ranks in the order of Section 2.2, so every list N+(x) holds only ranks > x
// and is sorted ascending.  For an edge u -> v, every common element w of the two lists is
// > v, so |N+(u) n N+(v)| = |suffix of N+(u) after v  n  N+(v)|.  The kernel therefore groups
// the work by the middle vertex v: N+(v) is staged once in LDS and the suffixes of the lists
// of all in-neighbours u of v are streamed through it.  The number of membership tests is
// sum_u C(d+(u), 2) instead of the sum of the lengths of both lists per edge; each test is
// one LDS bit lookup when N+(v) fits a bitmap over its rank range.
//
// Work items are (v, a chunk of v's in-edges).  One persistent kernel pulls items from two
// device counters: first the "workgroup" items (out-lists whose rank span needs the
// workgroup's whole LDS bitmap, or a sorted list), cooperatively, then the "wave" items, each
// wave with its own slice of LDS.  Items run heaviest (highest-rank) vertices first.  Inside a
// wave every in-edge suffix is cut into pieces of kPiece consecutive elements and each lane
// runs whole pieces, so one load and one lookup per element are the per-element costs,
// whatever the spread of suffix lengths.
//
// Panels.  Most of the tests sit at the highest ranks (the highest degrees), where a list N+(u)
// holds several consecutive middle vertices and its suffix would be streamed once for each.
// The top ranks are therefore grouped into panels of kPanel consecutive middle vertices
// P .. P + kPanel - 1: a panel's table M in LDS holds, for every rank w, the kPanel-bit mask
// of the panel vertices whose out-list contains w, and a segment is a pair (u, panel) with
// the mask R(u) of the panel vertices in N+(u).  Its suffix after the first of them is
// streamed once and each element w adds popcount(M[w] & R(u)): every panel vertex v with
// v in N+(u) and w in N+(v) closes one triangle (w > v holds because w is in N+(v)).
//
// Per-vertex counts (T(x) = triangles through x) use sorted lists in LDS instead of bitmaps
// so that a hit's position indexes an LDS counter: T(w) for the third vertex is flushed once
// per item, T(u) once per in-edge, T(v) once per item and wave.
#include <type_traits>

#include "internal.h"

namespace tc {

constexpr uint32_t kPiece = 16;
// pieces of the unmasked 16-bit probes (hcol rows carry the padding they need)
constexpr uint32_t kPieceHigh = 32;
constexpr int kThreads = 1024;
constexpr int kWgsPerCu = 1;  // workgroups per CU the LDS footprint allows
constexpr int kWaves = kThreads / kWave;
constexpr uint32_t kLdsWords = 32768;                 // 128 KiB per workgroup
constexpr uint32_t kSliceWords = kLdsWords / kWaves;  // 8 KiB per wave
constexpr uint32_t kWaveBits = kSliceWords * 32 - 32; // wave bitmap: span < 65504
constexpr uint32_t kWaveListPV = kSliceWords / 2;     // per-vertex: list + counters per wave
// per-vertex wave items with a bit filter: list, counters, filter and hit queue in a quarter of
// the slice each
constexpr uint32_t kFilterList = kSliceWords / 4;
constexpr uint32_t kFilterBits = kFilterList * 32;
constexpr uint32_t kHitQueue = kFilterList / 2;       // (entry, segment) pairs
// per-vertex counts: the highest ranks' credits as third vertices are summed in LDS per
// workgroup, in what LDS is left.  Nearly every wave item credits the very highest of them, and
// atomics on one address take 11 ns each, 2.7 ms for the 247,000 items at R-MAT 22.  Per-vertex
// counts at R-MAT 20, 21 and 23: 1.47, 3.25 and 30.4 ms before, 1.21, 2.79 and 28.4 with the sums
constexpr uint32_t kHotRanks = 768;
constexpr uint32_t kBlockBits = kLdsWords * 32 - 32;  // workgroup bitmap: span < 1048544
constexpr uint32_t kBlockList = kLdsWords;            // workgroup sorted list
constexpr uint32_t kBlockListPV = kLdsWords / 2;      // per-vertex: list + counters
constexpr uint32_t kItemEdgesWave = 512;     // default in-edges per wave item
constexpr uint32_t kItemEdgesBlock = 65536;  // default in-edges per workgroup item
constexpr uint32_t kPanel = 32;                       // one bit per panel vertex in a mask
constexpr uint32_t kPanelRanks = kLdsWords - 32;      // mask table: one word per rank
// per-vertex counts over a panel keep a third-vertex counter beside every mask word, so a
// panel's ranks are taken in windows of kPvWindow ranks, each with its table and counters in
// half of the workgroup's LDS (words 0 .. kPvWindow - 1, and word kPvWindow always zero)
constexpr uint32_t kPvPanelWords = kLdsWords / 2;
constexpr uint32_t kPvWindow = kPvPanelWords - 1;
// batched kernel: rows with at most kLightMax forward entries are counted edge by edge, at most
// kLightChunkMax staged entries at a time
constexpr uint32_t kLightMax = 256;
constexpr uint32_t kLightChunkMax = 1536;
// light rows' pieces: their lists are short (a few elements), so shorter pieces waste fewer
// lookups on masked positions
constexpr uint32_t kLightPiece = 8;
// middle-vertex kernels: a list with at most kLightList in-edges u -> v and at most that many
// entries in N+(v) is light.  A wave item costs about 560 vector instructions and a chain of
// loads whatever its size, and eight of them an atomic on the queue; with 8 in-edges of 8 entries
// each (a small-world graph of 1,000,003 vertices) that was nearly all of the counting kernel's
// 1.43 ms, and light lists take 0.14 + 0.03 ms.  R-MAT 23: 14.5 -> 13.1 + 0.2 ms.  Limits of 32
// and 128 measured slower at R-MAT 20 (2041 and 2353 us a count against 1960)
constexpr uint32_t kLightList = 64;
constexpr uint32_t kLightListWindow = 512;  // staged entries per wave
constexpr uint32_t kLightShiftMax = 4, kLightShiftMin = 2;  // lists per wave, log2 (light_shift)
constexpr int kLightThreads = 256;
constexpr int kLightWaves = kLightThreads / kWave;

// LDS access by byte address (32-bit LDS pointers)
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ uint32_t lds_word(uint32_t addr) {
    return *(const lds_u32 *)(uintptr_t)addr;
}
__device__ __forceinline__ uint32_t lds_addr(const uint32_t *p) {
    return (uint32_t)(uintptr_t)(const lds_u32 *)p;
}

// ------------------------------------------------------------------ membership probes

// N+(v) as a bitmap over ranks [lo, lo + span].  Bit span + 1 is always zero and lies inside
// the LDS region (spans are kept below the region's bits minus 32), so an id outside the span
// is clamped onto it instead of branching: every lookup is one unconditional LDS read.
struct BitmapProbe {
    const uint32_t *bm;
    uint32_t lo, span;
    __device__ __forceinline__ uint32_t bit(uint32_t w) const {
        const uint32_t o = min(w - lo, span + 1u);
        return __builtin_amdgcn_ubfe(bm[__builtin_amdgcn_ubfe(o, 5u, 27u)], o, 1u);
    }
    static constexpr bool kMasked = false;
    static constexpr bool kList = false;
    // totals streamer (run_batch_t): both parts of a segment, positions tested
    static constexpr bool kLow = true;
    static constexpr bool kMaskHigh = true;
    static constexpr bool kPanel = false;
};

// Panel table M over ranks [lo, lo + span]: word w - lo holds the mask of the panel vertices
// whose out-list contains w.  Word span + 1 is always zero, so out-of-range ids clamp onto it.
struct PanelProbe {
    const uint32_t *m;
    uint32_t lo, span;
    static constexpr bool kMasked = true;
    static constexpr bool kList = false;
    __device__ __forceinline__ uint32_t count(uint32_t w, uint32_t r) const {
        return __popc(m[min(w - lo, span + 1u)] & r);
    }
};

// A sorted list in LDS (d >= 1, uniform): the searches of a piece's kPiece entries advance in
// lockstep, three vector operations and one LDS read per step (byte addresses; the steps are the
// same for all lanes).  After search(), at[i] is the address of the last entry <= wv[i] (the
// list's start when none is) and bit kPiece - 1 - i of the result is set when it equals wv[i].
struct LdsListProbe {
    uint32_t list;  // LDS byte address
    uint32_t d;
    static constexpr bool kMasked = false;
    static constexpr bool kList = true;
    static constexpr bool kLow = true;
    static constexpr bool kMaskHigh = true;
    static constexpr bool kPanel = false;
    __device__ __forceinline__ uint32_t search(const uint32_t (&wv)[kPiece],
                                               uint32_t (&at)[kPiece]) const {
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i) at[i] = list;
        for (uint32_t left = (uint32_t)__builtin_amdgcn_readfirstlane((int)d); left > 1;) {
            const uint32_t half = left >> 1;
#pragma unroll
            for (uint32_t i = 0; i < kPiece; ++i) {
                const uint32_t mid = at[i] + half * 4u;
                at[i] = lds_word(mid) <= wv[i] ? mid : at[i];
            }
            left -= half;
        }
        uint32_t packed = 0;
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i)
            packed = packed + packed + (lds_word(at[i]) == wv[i] ? 1u : 0u);
        return packed;
    }
    // one entry per lane: the address of the last entry <= w
    __device__ __forceinline__ uint32_t search_one(uint32_t w) const {
        uint32_t at = list;
        for (uint32_t left = (uint32_t)__builtin_amdgcn_readfirstlane((int)d); left > 1;) {
            const uint32_t half = left >> 1, mid = at + half * 4u;
            at = lds_word(mid) <= w ? mid : at;
            left -= half;
        }
        return at;
    }
};

struct ListProbe {  // sorted list in global memory (d >= 1)
    const uint32_t *list;
    uint32_t d;
    static constexpr bool kMasked = false;
    static constexpr bool kList = true;
    static constexpr bool kLow = true;
    static constexpr bool kMaskHigh = true;
    static constexpr bool kPanel = false;
};

// ------------------------------------------------------------------ per-batch streaming

struct WaveScratch {  // tag: the segment's owner (per-vertex counts) or its panel mask, ...
    uint32_t off[kWave], beg[kWave], first[kWave], end[kWave], cnt[kWave], tag[kWave],
        aux[kWave];
};

// Segment sources: segment e is a range [b, en) of `col` streamed through the staged list,
// and `owner` is the vertex credited with the segment's hits in per-vertex counts.  rec(e)
// fetches everything a streamer needs of segment e at once.
struct SegRec {
    uint32_t b, en;  // the range of col
    uint32_t y;      // panel mask, or where the entries >= hbase start in col
    uint32_t h;      // where the entries >= hbase start in hcol
    uint32_t owner;
};

// In-edge records: the in-edge u -> v at CSR position e (list entry j holds cbeg[j] = e + 1)
// has its record at er[e] = (end of u's row, panel mask of u's run in a panel list or else
// where the suffix's entries >= hbase start in col, where they start in hcol, u); reading
// it is one random 16-byte gather per segment.  A panel's segment (u, panel) is the suffix of N+(u)
// after u's first panel vertex, tagged with the mask R(u) of u's panel vertices; with a high region
// every entry after a panel vertex is a rank >= p0 >= hbase.
struct InEdgeSegs {  // middle-vertex kernel: suffix of N+(u) after v, owner u
    const uint32_t *cbeg;
    const uint4 *er;
    __device__ __forceinline__ SegRec rec(uint32_t e) const {
        const uint32_t b = cbeg[e];
        const uint4 x = er[b - 1];
        return SegRec{b, x.x, x.y, x.z, x.w};
    }
};

struct OutEdgeSegs {  // u-centric kernel: the whole list N+(v) of out-neighbour v, owner v
    const uint2 *frow;
    const uint32_t *col;
    __device__ __forceinline__ SegRec rec(uint32_t e) const {
        const uint32_t v = col[e];
        const uint2 r = frow[v];
        return SegRec{r.x, r.y, 0u, 0u, v};
    }
};

// The calling wave streams segments [eb, min(eb + 64, e1)) of the current item through the
// probe and returns this lane's hits.  PV: per-vertex accumulation -- LDS counters `tcnt`
// indexed by the probe's position for a list in LDS, global atomics on `tpv` for one in memory;
// every segment's hits go to its owner.
template <bool PV, class Probe, class Segs>
__device__ __forceinline__ uint32_t run_batch(uint32_t eb, uint32_t e1, const Segs &segs,
                                              const uint32_t *__restrict__ col, const Probe &probe,
                                              WaveScratch &ws, uint32_t *tcnt,
                                              unsigned long long *__restrict__ tpv) {
    const uint32_t lane = lane_id();
    const uint32_t e = eb + lane;
    const bool valid = e < e1;
    SegRec r{0u, 0u, 0u, 0u, 0u};
    if (valid) r = segs.rec(e);
    const uint32_t b = r.b, en = r.en;
    // pieces are kPiece-element windows starting at 4-element (16-byte) boundaries, so a lane
    // reads its piece with kPiece / 4 aligned 16-byte loads; elements outside [b, en) are masked
    const uint32_t a0 = b & ~3u;
    const uint32_t p = (valid && en > b) ? (en - a0 + kPiece - 1) / kPiece : 0u;
    const uint32_t incl = wave_incl_scan(p);
    const uint32_t Q = wave_bcast(incl, kWave - 1);
    ws.off[lane] = incl - p;
    ws.beg[lane] = a0;
    ws.first[lane] = b;
    ws.end[lane] = en;
    if (PV) {
        ws.cnt[lane] = 0;
        ws.tag[lane] = r.owner;
    } else if (Probe::kMasked) {
        ws.tag[lane] = r.y;
    }
    wave_lds_sync();
    uint32_t hits_total = 0;
    for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
        const uint32_t q = q0 + lane;
        if (q < Q) {
            // owner: the last in-edge whose first piece is <= q (zero-piece lanes share the
            // offset of the next lane and lose to it)
            uint32_t k = 0;
#pragma unroll
            for (uint32_t step = 32; step; step >>= 1)
                if (ws.off[k + step] <= q) k += step;
            const uint32_t start = ws.beg[k] + (q - ws.off[k]) * kPiece;
            const uint32_t first = ws.first[k], stop = ws.end[k];
            const uint4 *p4 = reinterpret_cast<const uint4 *>(col + start);
            uint32_t wv[kPiece];
#pragma unroll
            for (uint32_t j = 0; j < kPiece / 4; ++j) {
                const uint4 x = p4[j];
                wv[4 * j] = x.x;
                wv[4 * j + 1] = x.y;
                wv[4 * j + 2] = x.z;
                wv[4 * j + 3] = x.w;
            }
            uint32_t hits = 0;
            if constexpr (!PV && Probe::kMasked) {
                // hits of element i: panel vertices of the owner whose lists hold it
                const uint32_t r = ws.tag[k];
                const uint32_t lo_i = first > start ? first - start : 0u;
                const uint32_t hi_i = min(stop - start, kPiece);
#pragma unroll
                for (uint32_t i = 0; i < kPiece; ++i) {
                    const uint32_t c = probe.count(wv[i], r);
                    hits += (i >= lo_i && i < hi_i) ? c : 0u;
                }
            } else if constexpr (std::is_same_v<Probe, LdsListProbe>) {
                // per-vertex counts credit the third vertex of every hit by its position
                uint32_t at[kPiece];
                const uint32_t found = probe.search(wv, at);
                const uint32_t lo_i = first > start ? first - start : 0u;
                const uint32_t hi_i = min(stop - start, kPiece);
                // (bit kPiece - 1 - i for entry i)
                const uint32_t packed = found & (((1u << kPiece) - 1u) >> lo_i) &
                                        ~((1u << (kPiece - hi_i)) - 1u);
                hits = __popc(packed);
                if (PV && packed) {
#pragma unroll
                    for (uint32_t i = 0; i < kPiece; ++i)
                        if ((packed >> (kPiece - 1 - i)) & 1u)
                            atomicAdd(&tcnt[(at[i] - probe.list) >> 2], 1u);
                }
            } else if constexpr (Probe::kList) {
                // a list in memory:
                // the piece's 16 lookups as binary searches in lockstep (the list length is
                // uniform), so that every step issues independent reads; position pos is the
                // first entry >= w, and w is in the list iff that entry equals w.  Per-vertex
                // counts credit the third vertex of every hit.
                uint32_t base[kPiece];
#pragma unroll
                for (uint32_t i = 0; i < kPiece; ++i) base[i] = 0;
                for (uint32_t n_left = probe.d; n_left > 1;) {
                    const uint32_t half = n_left >> 1;
#pragma unroll
                    for (uint32_t i = 0; i < kPiece; ++i)
                        base[i] = probe.list[base[i] + half - 1] < wv[i] ? base[i] + half : base[i];
                    n_left -= half;
                }
                uint32_t packed = 0;
#pragma unroll
                for (uint32_t i = 0; i < kPiece; ++i) {
                    base[i] += probe.list[base[i]] < wv[i] ? 1u : 0u;
                    packed |= (probe.list[min(base[i], probe.d - 1u)] == wv[i] ? 1u : 0u) << i;
                }
                const uint32_t lo_i = first > start ? first - start : 0u;
                const uint32_t hi_i = min(stop - start, kPiece);
                const uint32_t hmask = hi_i >= 32u ? ~0u : ((1u << hi_i) - 1u);
                packed &= hmask & ~((1u << lo_i) - 1u);
                hits = __popc(packed);
                if (PV && packed) {
#pragma unroll
                    for (uint32_t i = 0; i < kPiece; ++i) {
                        if ((packed >> i) & 1u) atomicAdd(&tpv[wv[i]], 1ull);
                    }
                }
            } else {  // a bitmap
                static_assert(!PV, "per-vertex counts need positions");
                // the piece's valid elements are the contiguous range [lo_i, hi_i) of positions
                uint32_t packed = 0;
#pragma unroll
                for (uint32_t i = 0; i < kPiece; ++i) packed |= probe.bit(wv[i]) << i;
                const uint32_t lo_i = first > start ? first - start : 0u;
                const uint32_t hi_i = min(stop - start, kPiece);
                const uint32_t hmask = hi_i >= 32u ? ~0u : ((1u << hi_i) - 1u);
                const uint32_t mask = hmask & ~((1u << lo_i) - 1u);
                hits = __popc(packed & mask);
            }
            hits_total += hits;
            if (PV && hits) atomicAdd(&ws.cnt[k], hits);
        }
    }
    wave_lds_sync();
    if (PV) {
        if (ws.cnt[lane]) atomicAdd(&tpv[ws.tag[lane]], (unsigned long long)ws.cnt[lane]);
        wave_lds_sync();
    }
    return hits_total;
}

// ------------------------------------------------------------------ totals streaming
//
// Total counts stream a segment in two parts: its entries below rank hbase from col (32-bit
// pieces of kPiece entries from 4-aligned positions), and its entries >= hbase from hcol as
// 16-bit offsets from hbase (pieces of kPiece, or kPieceHigh for unmasked probes, entries from
// 8-aligned positions).  In hcol every row's part starts at an 8-aligned position and is
// followed by zeros up to the next multiple of 8 and kPieceHigh - 8 more, so a piece never
// reaches another row.
//
// Masked probes test only the entries inside the segment.  Unmasked probes test every entry
// of a piece: the entries of u's row before the segment are ranks up to the middle vertex
// (or up to u's first panel vertex), and the padding zeros stand for rank hbase; the probes
// below are built so that none of these can hit.

// Bitmap over the whole high region: bit x for rank hbase + x (x < 2^16, the wave's LDS
// slice).  For middle vertices v >= hbase only: N+(v) lies in (v, n), so neither a rank <= v
// nor hbase is ever set.
struct HighBitmapProbe {
    uint32_t base;  // LDS byte address of the slice: a multiple of its 8 KiB
    static constexpr bool kLow = false;
    static constexpr bool kMaskHigh = false;
    static constexpr bool kPanel = false;
    // bits of the two entries of a packed pair of 16-bit entries: word x >> 5 is at byte
    // ((x >> 3) & 0x1ffc) | base, and the bit offset of v_bfe is the low 5 bits of its
    // operand, so the low entry needs no extraction
    __device__ __forceinline__ uint32_t bit_lo(uint32_t pr) const {
        return __builtin_amdgcn_ubfe(lds_word(((pr >> 3) & 0x1ffcu) | base), pr, 1u);
    }
    __device__ __forceinline__ uint32_t bit_hi(uint32_t pr) const {
        return __builtin_amdgcn_ubfe(lds_word(((pr >> 19) & 0x1ffcu) | base), pr >> 16, 1u);
    }
    __device__ __forceinline__ uint32_t bits2(uint32_t pr) const { return bit_lo(pr) + bit_hi(pr); }
};

// The entries >= hbase of N+(v) for a middle vertex below hbase (a rank span too wide for a
// bitmap) in a high-region bitmap (as HighBitmapProbe), for the 16-bit pieces only.  Masked:
// such a suffix's high part starts at its row's part of hcol, but the padding zeros (rank
// hbase) may be in N+(v).
struct HighMaskedProbe {
    HighBitmapProbe hi;
    static constexpr bool kLow = true;  // the segments have 32-bit parts (not streamed here)
    static constexpr bool kMaskHigh = true;
    static constexpr bool kPanel = false;
};

// Both in one pass, with the entries of N+(v) below hbase as a sorted list (1 to kWave entries, in
// the wave's scratch).
struct LowHighProbe {
    LdsListProbe low;
    HighMaskedProbe high;
    static constexpr bool kLow = true;
    static constexpr bool kMaskHigh = true;
    static constexpr bool kPanel = false;
};

// Panel table over ranks [P, n) (as PanelProbe) read with 16-bit entries: rank hbase + x is
// word x - c (c = P - hbase), ranks below P saturate onto word 0 (rank P, in no out-list of
// the panel), and no entry exceeds word n - 1 - P.  An entry of u's row up to u's first panel
// vertex P + j only matches panel vertices below P + j, none of which is in u's mask.
struct PanelHighProbe {
    const uint32_t *m;
    uint32_t c;
    static constexpr bool kLow = false;
    static constexpr bool kMaskHigh = false;
    static constexpr bool kPanel = true;
    __device__ __forceinline__ uint32_t count(uint32_t x, uint32_t r) const {
        const uint32_t o = x > c ? x - c : 0u;
        return __popc(m[o] & r);
    }
};

// bit i set when position start + i of a piece lies in [first, stop) (start < stop)
__device__ __forceinline__ uint32_t piece_mask(uint32_t start, uint32_t first, uint32_t stop) {
    const uint32_t lo_i = first > start ? first - start : 0u;
    const uint32_t hi_i = min(stop - start, kPiece);
    const uint32_t hmask = hi_i >= 32u ? ~0u : ((1u << hi_i) - 1u);
    return hmask & ~((1u << lo_i) - 1u);
}

// hits of the entries wv[i] at positions start + i that lie in [first, stop)
template <class Probe>
__device__ __forceinline__ uint32_t masked_hits(const Probe &probe, const uint32_t (&wv)[kPiece],
                                                uint32_t start, uint32_t first, uint32_t stop) {
    const uint32_t mask = piece_mask(start, first, stop);
    uint32_t packed = 0;
    if constexpr (std::is_same_v<Probe, LdsListProbe>) {
        uint32_t at[kPiece];
        // (bit kPiece - 1 - i for entry i)
        return __popc(probe.search(wv, at) & (__brev(mask) >> (32u - kPiece)));
    } else if constexpr (Probe::kList) {
        // the piece's lookups as binary searches in lockstep (the list length is uniform)
        uint32_t base[kPiece];
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i) base[i] = 0;
        for (uint32_t n_left = probe.d; n_left > 1;) {
            const uint32_t half = n_left >> 1;
#pragma unroll
            for (uint32_t i = 0; i < kPiece; ++i)
                base[i] = probe.list[base[i] + half - 1] < wv[i] ? base[i] + half : base[i];
            n_left -= half;
        }
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i) {
            base[i] += probe.list[base[i]] < wv[i] ? 1u : 0u;
            packed |= (probe.list[min(base[i], probe.d - 1u)] == wv[i] ? 1u : 0u) << i;
        }
    } else {
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i) packed |= probe.bit(wv[i]) << i;
    }
    return __popc(packed & mask);
}

// Piece evaluations of the totals streamer.  Masked probes: a 32-bit piece (entries wv) and a
// 16-bit piece (packed pairs pr of offsets from hbase), positions start + i, counted inside
// [first, stop).  Unmasked probes: a 16-bit piece of kPieceHigh entries, all counted.
template <class Probe>
__device__ __forceinline__ uint32_t low_hits(const Probe &probe, const uint32_t (&wv)[kPiece],
                                             uint32_t start, uint32_t first, uint32_t stop) {
    return masked_hits(probe, wv, start, first, stop);
}
template <class Probe>
__device__ __forceinline__ uint32_t high_hits(const Probe &probe,
                                              const uint32_t (&pr)[kPiece / 2], uint32_t hbase,
                                              uint32_t start, uint32_t first, uint32_t stop) {
    uint32_t wv[kPiece];
#pragma unroll
    for (uint32_t i = 0; i < kPiece / 2; ++i) {
        wv[2 * i] = hbase + (pr[i] & 0xFFFFu);
        wv[2 * i + 1] = hbase + (pr[i] >> 16);
    }
    return masked_hits(probe, wv, start, first, stop);
}
__device__ __forceinline__ uint32_t high_hits(const HighMaskedProbe &probe,
                                              const uint32_t (&pr)[kPiece / 2], uint32_t,
                                              uint32_t start, uint32_t first, uint32_t stop) {
    uint32_t packed = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPiece / 2; ++i)
        packed |= (probe.hi.bit_lo(pr[i]) << (2 * i)) | (probe.hi.bit_hi(pr[i]) << (2 * i + 1));
    return __popc(packed & piece_mask(start, first, stop));
}
__device__ __forceinline__ uint32_t high_hits_u(const HighBitmapProbe &probe,
                                                const uint32_t (&pr)[kPieceHigh / 2], uint32_t) {
    uint32_t hits = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPieceHigh / 2; ++i) hits += probe.bits2(pr[i]);
    return hits;
}
__device__ __forceinline__ uint32_t high_hits_u(const PanelHighProbe &probe,
                                                const uint32_t (&pr)[kPieceHigh / 2], uint32_t r) {
    uint32_t hits = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPieceHigh / 2; ++i)
        hits += probe.count(pr[i] & 0xFFFFu, r) + probe.count(pr[i] >> 16, r);
    return hits;
}

__device__ __forceinline__ uint32_t low_hits(const LowHighProbe &probe,
                                             const uint32_t (&wv)[kPiece], uint32_t start,
                                             uint32_t first, uint32_t stop) {
    return low_hits(probe.low, wv, start, first, stop);
}
__device__ __forceinline__ uint32_t high_hits(const LowHighProbe &probe,
                                              const uint32_t (&pr)[kPiece / 2], uint32_t hbase,
                                              uint32_t start, uint32_t first, uint32_t stop) {
    return high_hits(probe.high, pr, hbase, start, first, stop);
}

// The calling wave streams one batch of up to 64 segments (r: this lane's record, all zero
// for no segment) through the probe for total counts and returns this lane's hits.  A segment
// is the col range [b, en) whose entries from hb on are ranks >= hbase, found in hcol from
// position h; probes without kLow are only given segments with hb == b.  The batch's 32-bit
// pieces (of [b, hb)) run first, then its 16-bit pieces, each as its own sequence of rounds,
// so that a round holds pieces of one kind.
template <class Probe, int kParts = 3>
__device__ __forceinline__ uint32_t run_batch_t(const SegRec &r,
                                                const uint32_t *__restrict__ col,
                                                const uint16_t *__restrict__ hcol,
                                                uint32_t hbase, const Probe &probe,
                                                WaveScratch &ws) {
    const uint32_t lane = lane_id();
    // panel segments are high throughout; other segments switch to high entries at r.y
    const uint32_t b = r.b, en = r.en, h = r.h;
    const uint32_t hb = Probe::kPanel ? b : r.y;
    const uint32_t a0 = b & ~3u;
    const uint32_t pl = (Probe::kLow && hb > b) ? (hb - a0 + kPiece - 1) / kPiece : 0u;
    // unmasked probes read longer pieces (the per-piece search and setup is their overhead)
    constexpr uint32_t kPh = Probe::kMaskHigh ? kPiece : kPieceHigh;
    const uint32_t hl = en - hb;
    const uint32_t ph = hl ? (h + hl - (h & ~7u) + kPh - 1) / kPh : 0u;
    static_assert(kParts >= 1 && kParts <= 3, "kParts: 1 the 32-bit pieces, 2 the 16-bit ones");
    ws.off[lane] = 0u;  // the rounds' marker table
    ws.aux[lane] = h;
    if constexpr (Probe::kLow) {
        ws.beg[lane] = a0;
        ws.first[lane] = b;
        ws.end[lane] = hb;
    }
    if constexpr (Probe::kMaskHigh) ws.tag[lane] = h + hl;
    if constexpr (Probe::kPanel) ws.tag[lane] = r.y;
    uint32_t hits_total = 0, carry = 0, round = 0;
    if constexpr (Probe::kLow && (kParts & 1)) {  // the 32-bit pieces
        const uint32_t incl = wave_incl_scan(pl);
        const uint32_t Q = wave_bcast(incl, kWave - 1);
        const uint32_t my_off = incl - pl;
        wave_lds_sync();
        for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
            const uint32_t k = round_owner(ws.off, my_off, pl, q0, ++round, carry) - 1u;
            const uint32_t off_k = wave_bcast_from(my_off, k);
            const uint32_t q = q0 + lane;
            if (q < Q) {
                const uint32_t start = ws.beg[k] + (q - off_k) * kPiece;
                const uint4 *p4 = reinterpret_cast<const uint4 *>(col + start);
                uint32_t wv[kPiece];
#pragma unroll
                for (uint32_t i = 0; i < kPiece / 4; ++i) {
                    const uint4 x = p4[i];
                    wv[4 * i] = x.x;
                    wv[4 * i + 1] = x.y;
                    wv[4 * i + 2] = x.z;
                    wv[4 * i + 3] = x.w;
                }
                hits_total += low_hits(probe, wv, start, ws.first[k], ws.end[k]);
            }
        }
        carry = 0;
    }
    if constexpr ((kParts & 2) != 0) {  // the 16-bit pieces
        const uint32_t incl = wave_incl_scan(ph);
        const uint32_t Q = wave_bcast(incl, kWave - 1);
        const uint32_t my_off = incl - ph;
        wave_lds_sync();
        for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
            const uint32_t k = round_owner(ws.off, my_off, ph, q0, ++round, carry) - 1u;
            const uint32_t off_k = wave_bcast_from(my_off, k);
            const uint32_t q = q0 + lane;
            if (q < Q) {
                const uint32_t hs = ws.aux[k];
                const uint32_t start = (hs & ~7u) + (q - off_k) * kPh;
                const uint4 *p4 = reinterpret_cast<const uint4 *>(hcol + start);
                uint32_t pr[kPh / 2];
#pragma unroll
                for (uint32_t i = 0; i < kPh / 8; ++i) {
                    const uint4 x = p4[i];
                    pr[4 * i] = x.x;
                    pr[4 * i + 1] = x.y;
                    pr[4 * i + 2] = x.z;
                    pr[4 * i + 3] = x.w;
                }
                if constexpr (Probe::kMaskHigh)
                    hits_total += high_hits(probe, pr, hbase, start, hs, ws.tag[k]);
                else
                    hits_total += high_hits_u(probe, pr, ws.tag[k]);
            }
        }
    }
    wave_lds_sync();
    return hits_total;
}

// The calling wave streams the segments first, first + step, ... (its batches of 64: lanes
// take consecutive segments) of an item ending at e1 for total counts.  (Fetching the
// records a batch or two ahead measured no faster: the gathers' lines, not their latency,
// are the cost.)
template <int kParts = 3, class Probe, class Segs>
__device__ __forceinline__ uint32_t stream_t(uint32_t first, uint32_t e1, uint32_t step,
                                             const Segs &segs,
                                             const uint32_t *__restrict__ col,
                                             const uint16_t *__restrict__ hcol, uint32_t hbase,
                                             const Probe &probe, WaveScratch &ws) {
    const uint32_t lane = lane_id();
    uint32_t hits = 0;
    for (uint32_t eb = first; eb < e1; eb += step) {
        const SegRec r = eb + lane < e1 ? segs.rec(eb + lane) : SegRec{0u, 0u, 0u, 0u, 0u};
        hits += run_batch_t<Probe, kParts>(r, col, hcol, hbase, probe, ws);
    }
    return hits;
}

// Wave-private claims on a shared item counter: `claim` consecutive positions per atomic, so
// that the counter (one address that every XCD's waves update) sees few operations when items
// are small.  Items are sorted heaviest first, so a claim holds items of similar size.
struct WaveQueue {
    uint32_t claim, next = 0, end = 0;
    __device__ __forceinline__ bool pop(uint32_t *counter, uint32_t n_items, uint32_t &q) {
        if (next == end) {
            // (No claim on an empty queue: 4096 waves' atomics on one address take 45 us, 11 ns each.
            // A load of the counter before the claims that may fail costs as much as an atomic while
            // others claim.  With a look near the queue's end and without, a resident graph: 600
            // cliques of 130 vertices 383 and 288 us, R-MAT 20 634 and 609, R-MAT 21 1497 and 1314.)
            uint32_t c = n_items;
            if (lane_id() == 0 && n_items) c = atomicAdd(counter, claim);
            c = wave_bcast(c, 0);
            if (c >= n_items) return false;
            next = c;
            end = min(c + claim, n_items);
        }
        q = next++;
        return true;
    }
};
constexpr uint32_t kClaimWave = 8;      // middle-vertex kernel, wave items
constexpr uint32_t kClaimBatched = 64;  // batched kernel, heavy items: at most

struct ItemRange {
    uint32_t v, e0, e1, r0, d;
};

// Item q of a queue covers in-edges [e0, e1) of list c = row block * (n + 1) + v.
__device__ __forceinline__ ItemRange item_range(uint32_t q, uint32_t kitem, uint32_t n1,
                                                const uint32_t *__restrict__ item_c,
                                                const uint32_t *__restrict__ item_off,
                                                const uint32_t *__restrict__ cptr,
                                                const uint32_t *__restrict__ row_ptr) {
    ItemRange it;
    const uint32_t c = item_c[q];
    it.v = c % n1;
    const uint32_t chunk = q - item_off[c];
    it.e0 = cptr[c] + chunk * kitem;
    it.e1 = min(it.e0 + kitem, cptr[c + 1]);
    it.r0 = row_ptr[it.v];
    it.d = row_ptr[it.v + 1] - it.r0;
    return it;
}

// ------------------------------------------------------------------ per-vertex panels
//
// Per-vertex counts over a panel P .. P+31 in one pass, with the panel table of the totals.
// Element w of segment (u, panel) closes one triangle u -> P+j -> w for every bit j of
// c = M[w] & R(u); each is credited three times:
//   the first vertex u: popcount(c), summed per segment (one atomic per segment);
//   the third vertex w: popcount(c) into an LDS counter beside M[w] (flushed once per item);
//   the middle vertex P+j: bit j of c, summed per lane in bit-sliced counters (bit j of
//   plane k is bit k of the count of panel vertex j), with a carry-save adder tree over the
//   16 elements of a piece, and flushed once per item.

// carry-save adder: (h, l) with 2h + l = l + b + c bitwise
__device__ __forceinline__ void csa(uint32_t &h, uint32_t &l, uint32_t b, uint32_t c) {
    const uint32_t u = l ^ b;
    h = (l & b) | (u & c);
    l = u ^ c;
}

// 32 counters (one per panel vertex) of one lane in bit slices: the count of vertex j is
// ones_j + 2 twos_j + 4 fours_j + 8 eights_j + 16 * (sum_k hi[k]_j 2^k)
struct MidCounters {
    // counts up to 4095 per lane between flushes: a flush every 255 pieces costs a few percent
    // of the pieces' work, and the largest panels reach it (the flush path runs in practice)
    static constexpr int kHi = 8;
    uint32_t ones, twos, fours, eights, hi[kHi];
    __device__ __forceinline__ void clear() {
        ones = twos = fours = eights = 0;
#pragma unroll
        for (int k = 0; k < kHi; ++k) hi[k] = 0;
    }
    // adds the 16 masks d[0..15] (Harley-Seal tree)
    __device__ __forceinline__ void add16(const uint32_t (&d)[16]) {
        uint32_t tA, tB, fA, fB, eA, eB, sx;
        csa(tA, ones, d[0], d[1]);
        csa(tB, ones, d[2], d[3]);
        csa(fA, twos, tA, tB);
        csa(tA, ones, d[4], d[5]);
        csa(tB, ones, d[6], d[7]);
        csa(fB, twos, tA, tB);
        csa(eA, fours, fA, fB);
        csa(tA, ones, d[8], d[9]);
        csa(tB, ones, d[10], d[11]);
        csa(fA, twos, tA, tB);
        csa(tA, ones, d[12], d[13]);
        csa(tB, ones, d[14], d[15]);
        csa(fB, twos, tA, tB);
        csa(eB, fours, fA, fB);
        csa(sx, eights, eA, eB);
        uint32_t carry = sx;
#pragma unroll
        for (int k = 0; k < kHi; ++k) {
            const uint32_t t = hi[k] & carry;
            hi[k] ^= carry;
            carry = t;
        }
    }
    __device__ __forceinline__ uint32_t count(uint32_t j) const {
        uint32_t h = 0;
#pragma unroll
        for (int k = kHi - 1; k >= 0; --k) h = (h << 1) | ((hi[k] >> j) & 1u);
        return ((ones >> j) & 1u) + 2u * ((twos >> j) & 1u) + 4u * ((fours >> j) & 1u) +
               8u * ((eights >> j) & 1u) + 16u * h;
    }
    // wave sums into the workgroup's 32 middle-vertex counters, then restart
    __device__ __forceinline__ void flush(unsigned long long *mid) {
#pragma unroll 1
        for (uint32_t j = 0; j < kPanel; ++j) {
            const uint64_t s = wave_sum_u64(count(j));
            if (lane_id() == 0 && s) atomicAdd(&mid[j], (unsigned long long)s);
        }
        clear();
    }
};
// pieces one lane may add between flushes (16 per piece per counter, kHi + 4 bits)
constexpr uint32_t kMidPieces = (1u << (MidCounters::kHi + 4)) / kPiece - 1;

// The calling wave streams panel segments [eb, min(eb + 64, e1)) of the current item through
// the mask table m (and third-vertex counters cnt3 at the same offsets) and returns this
// lane's hits; `pieces` is the wave's bound on the pieces any lane added to mc since its last
// flush.
__device__ __forceinline__ uint32_t run_panel_pv(uint32_t eb, uint32_t e1,
                                                 const InEdgeSegs &segs,
                                                 const uint32_t *__restrict__ col,
                                                 const uint32_t *m, uint32_t *cnt3, uint32_t lo,
                                                 uint32_t span, WaveScratch &ws,
                                                 MidCounters &mc, uint32_t &pieces,
                                                 unsigned long long *mid,
                                                 unsigned long long *__restrict__ tpv) {
    const uint32_t lane = lane_id();
    const uint32_t e = eb + lane;
    const bool valid = e < e1;
    SegRec r{0u, 0u, 0u, 0u, 0u};
    if (valid) r = segs.rec(e);
    const uint32_t b = r.b, en = r.en;
    const uint32_t a0 = b & ~3u;
    const uint32_t p = (valid && en > b) ? (en - a0 + kPiece - 1) / kPiece : 0u;
    const uint32_t incl = wave_incl_scan(p);
    const uint32_t Q = wave_bcast(incl, kWave - 1);
    ws.off[lane] = incl - p;
    ws.beg[lane] = a0;
    ws.first[lane] = b;
    ws.end[lane] = en;
    ws.cnt[lane] = 0;
    ws.tag[lane] = r.y;      // the panel mask R(u)
    ws.aux[lane] = r.owner;  // u
    wave_lds_sync();
    const uint32_t per_lane = (Q + kWave - 1) / kWave;
    if (pieces + per_lane > kMidPieces) {
        mc.flush(mid);
        pieces = 0;
    }
    pieces += per_lane;
    uint32_t hits_total = 0;
    for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
        const uint32_t q = q0 + lane;
        uint32_t c[kPiece];
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i) c[i] = 0;
        if (q < Q) {
            uint32_t k = 0;
#pragma unroll
            for (uint32_t step = 32; step; step >>= 1)
                if (ws.off[k + step] <= q) k += step;
            const uint32_t start = ws.beg[k] + (q - ws.off[k]) * kPiece;
            const uint32_t first = ws.first[k], stop = ws.end[k];
            const uint4 *p4 = reinterpret_cast<const uint4 *>(col + start);
            uint32_t wv[kPiece];
#pragma unroll
            for (uint32_t j = 0; j < kPiece / 4; ++j) {
                const uint4 x = p4[j];
                wv[4 * j] = x.x;
                wv[4 * j + 1] = x.y;
                wv[4 * j + 2] = x.z;
                wv[4 * j + 3] = x.w;
            }
            const uint32_t r = ws.tag[k];
            const uint32_t lo_i = first > start ? first - start : 0u;
            const uint32_t hi_i = min(stop - start, kPiece);
            uint32_t hits = 0;
#pragma unroll
            for (uint32_t i = 0; i < kPiece; ++i) {
                // an id outside the table clamps onto word span + 1, which is always zero
                const uint32_t o = min(wv[i] - lo, span + 1u);
                const uint32_t ci = (i >= lo_i && i < hi_i) ? (m[o] & r) : 0u;
                c[i] = ci;
                const uint32_t h = __popc(ci);
                hits += h;
                if (h) atomicAdd(&cnt3[o], h);
            }
            hits_total += hits;
            if (hits) atomicAdd(&ws.cnt[k], hits);
        }
        mc.add16(c);
    }
    wave_lds_sync();
    if (ws.cnt[lane]) atomicAdd(&tpv[ws.aux[lane]], (unsigned long long)ws.cnt[lane]);
    wave_lds_sync();
    return hits_total;
}

// Per-vertex wave items with N+(v) of at most kFilterList entries.  Nearly every entry streamed
// is no hit, and a lockstep search costs log2(d) LDS reads and three times that many vector
// operations per entry: at R-MAT 22, 800 LDS and 2,780 vector instructions per item.  So the
// slice also holds a filter, bit w mod kFilterBits of every w in N+(v): one read per entry passes
// the hits and d in kFilterBits of the others.  The entries passed are queued with their segments,
// and every lane searches one of them per step (290 and 1,500 instructions).  A round that passes
// more entries than the queue holds is searched in lockstep.  Longer lists (0.3 percent of the
// items at R-MAT 22) keep the lockstep search: the slice has no room for more.  Per-vertex counts,
// R-MAT 22 with the preprocessing 11.05 -> 10.37 ms, R-MAT 23 without 28.4 -> 25.3 ms; bound by
// missed lines now (3.9 TB/s at R-MAT 22).
// mem: list, counters, filter (zero but for N+(v)'s bits) and queue.
__device__ __forceinline__ uint32_t run_filter_pv(uint32_t eb, uint32_t e1,
                                                  const InEdgeSegs &segs,
                                                  const uint32_t *__restrict__ col,
                                                  uint32_t *mem, uint32_t d, WaveScratch &ws,
                                                  unsigned long long *__restrict__ tpv) {
    const uint32_t lane = lane_id();
    uint32_t *tc = mem + kFilterList;
    const uint32_t *filter = mem + 2 * kFilterList;
    uint2 *queue = reinterpret_cast<uint2 *>(mem + 3 * kFilterList);
    const LdsListProbe probe{lds_addr(mem), d};
    const SegRec r = eb + lane < e1 ? segs.rec(eb + lane) : SegRec{0u, 0u, 0u, 0u, 0u};
    const uint32_t a0 = r.b & ~3u;
    const uint32_t p = r.en > r.b ? (r.en - a0 + kPiece - 1) / kPiece : 0u;
    const uint32_t incl = wave_incl_scan(p);
    const uint32_t Q = wave_bcast(incl, kWave - 1);
    const uint32_t my_off = incl - p;
    ws.off[lane] = 0u;  // the rounds' marker table
    ws.beg[lane] = a0;
    ws.first[lane] = r.b;
    ws.end[lane] = r.en;
    ws.cnt[lane] = 0u;
    ws.tag[lane] = r.owner;
    wave_lds_sync();
    uint32_t hits = 0, carry = 0, round = 0;
    for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
        const uint32_t k = round_owner(ws.off, my_off, p, q0, ++round, carry) - 1u;
        const uint32_t off_k = wave_bcast_from(my_off, k);
        const uint32_t q = q0 + lane;
        uint32_t wv[kPiece];
#pragma unroll
        for (uint32_t i = 0; i < kPiece; ++i) wv[i] = 0u;
        uint32_t packed = 0;  // bit kPiece - 1 - i for entry i
        if (q < Q) {
            const uint32_t start = ws.beg[k] + (q - off_k) * kPiece;
            const uint32_t first = ws.first[k], stop = ws.end[k];
            const uint4 *p4 = reinterpret_cast<const uint4 *>(col + start);
#pragma unroll
            for (uint32_t j = 0; j < kPiece / 4; ++j) {
                const uint4 x = p4[j];
                wv[4 * j] = x.x;
                wv[4 * j + 1] = x.y;
                wv[4 * j + 2] = x.z;
                wv[4 * j + 3] = x.w;
            }
#pragma unroll
            for (uint32_t i = 0; i < kPiece; ++i)
                packed = packed + packed +
                         __builtin_amdgcn_ubfe(filter[(wv[i] & (kFilterBits - 1u)) >> 5], wv[i],
                                               1u);
            const uint32_t lo_i = first > start ? first - start : 0u;
            const uint32_t hi_i = min(stop - start, kPiece);
            packed &= (((1u << kPiece) - 1u) >> lo_i) & ~((1u << (kPiece - hi_i)) - 1u);
        }
        const uint32_t np = (uint32_t)__popc(packed);
        const uint32_t upto = wave_incl_scan(np);
        const uint32_t passed = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
        if (passed <= kHitQueue) {
            uint32_t at = upto - np;
#pragma unroll
            for (uint32_t i = 0; i < kPiece; ++i)
                if ((packed >> (kPiece - 1 - i)) & 1u) queue[at++] = make_uint2(wv[i], k);
            wave_lds_sync();
            for (uint32_t j = lane; j < passed; j += kWave) {
                const uint2 x = queue[j];
                const uint32_t pos = probe.search_one(x.x);
                if (lds_word(pos) == x.x) {
                    ++hits;
                    atomicAdd(&tc[(pos - probe.list) >> 2], 1u);
                    atomicAdd(&ws.cnt[x.y], 1u);
                }
            }
            wave_lds_sync();
        } else {
            uint32_t at[kPiece];
            packed &= probe.search(wv, at);
            if (packed) {
                hits += (uint32_t)__popc(packed);
                atomicAdd(&ws.cnt[k], (uint32_t)__popc(packed));
#pragma unroll
                for (uint32_t i = 0; i < kPiece; ++i)
                    if ((packed >> (kPiece - 1 - i)) & 1u)
                        atomicAdd(&tc[(at[i] - probe.list) >> 2], 1u);
            }
        }
    }
    wave_lds_sync();
    if (ws.cnt[lane]) atomicAdd(&tpv[ws.tag[lane]], (unsigned long long)ws.cnt[lane]);
    wave_lds_sync();
    return hits;
}

// first position in hcol[b, e) (ascending) whose entry is >= x
__device__ __forceinline__ uint32_t hcol_lower_bound(const uint16_t *__restrict__ hcol,
                                                     uint32_t b, uint32_t e, uint32_t x) {
    while (b < e) {
        const uint32_t mid = b + ((e - b) >> 1);
        if (hcol[mid] < x) b = mid + 1;
        else e = mid;
    }
    return b;
}

// The same for panels in the high region: every suffix entry is read from hcol as a 16-bit
// offset from hbase, in unmasked pieces of kPieceHigh entries (entries of u's row up to its
// first panel vertex only match panel vertices below it, none of which is in its mask, and
// padding zeros, rank hbase, lie below the window; entries outside the window clamp onto the
// zero word), with the owners found as in the totals streamer.  The window's table covers
// offsets [c, c + wn) from hbase; with cut_lo / cut_hi the segment's entries below / above
// the window are found by a binary search and not streamed.
__device__ __forceinline__ uint32_t run_panel_pv_high(const SegRec &r,
                                                      const uint16_t *__restrict__ hcol,
                                                      const uint32_t *m, uint32_t *cnt3,
                                                      uint32_t c, uint32_t wn, bool cut_lo,
                                                      bool cut_hi, WaveScratch &ws,
                                                      MidCounters &mc, uint32_t &pieces,
                                                      unsigned long long *mid,
                                                      unsigned long long *__restrict__ tpv) {
    const uint32_t lane = lane_id();
    uint32_t h0 = r.h, h1 = r.h + (r.en - r.b);
    if (h1 > h0 && cut_lo) h0 = hcol_lower_bound(hcol, h0, h1, c);
    if (h1 > h0 && cut_hi) h1 = hcol_lower_bound(hcol, h0, h1, c + wn);
    const uint32_t hl = h1 > h0 ? h1 - h0 : 0u, h = h0;
    const uint32_t ph = hl ? (h + hl - (h & ~7u) + kPieceHigh - 1) / kPieceHigh : 0u;
    ws.off[lane] = 0u;  // the rounds' marker table
    ws.aux[lane] = h;
    ws.tag[lane] = r.y;      // the panel mask R(u)
    ws.beg[lane] = r.owner;  // u
    ws.cnt[lane] = 0u;
    const uint32_t incl = wave_incl_scan(ph);
    const uint32_t Q = wave_bcast(incl, kWave - 1);
    const uint32_t my_off = incl - ph;
    wave_lds_sync();
    // a piece adds kPieceHigh / kPiece groups of kPiece masks to the middle-vertex counters
    const uint32_t per_lane = (Q + kWave - 1) / kWave * (kPieceHigh / kPiece);
    if (pieces + per_lane > kMidPieces) {
        mc.flush(mid);
        pieces = 0;
    }
    pieces += per_lane;
    uint32_t hits_total = 0, carry = 0, round = 0;
    for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
        const uint32_t k = round_owner(ws.off, my_off, ph, q0, ++round, carry) - 1u;
        const uint32_t off_k = wave_bcast_from(my_off, k);
        const uint32_t q = q0 + lane;
        uint32_t cm[kPieceHigh];
#pragma unroll
        for (uint32_t i = 0; i < kPieceHigh; ++i) cm[i] = 0;
        if (q < Q) {
            const uint32_t start = (ws.aux[k] & ~7u) + (q - off_k) * kPieceHigh;
            const uint4 *p4 = reinterpret_cast<const uint4 *>(hcol + start);
            uint32_t pr[kPieceHigh / 2];
#pragma unroll
            for (uint32_t i = 0; i < kPieceHigh / 8; ++i) {
                const uint4 x = p4[i];
                pr[4 * i] = x.x;
                pr[4 * i + 1] = x.y;
                pr[4 * i + 2] = x.z;
                pr[4 * i + 3] = x.w;
            }
            const uint32_t rm = ws.tag[k];
            uint32_t hits = 0;
#pragma unroll
            for (uint32_t i = 0; i < kPieceHigh; ++i) {
                const uint32_t x = (i & 1u) ? (pr[i >> 1] >> 16) : (pr[i >> 1] & 0xFFFFu);
                const uint32_t o = min(x - c, wn);  // outside the window: the zero word
                const uint32_t ci = m[o] & rm;
                cm[i] = ci;
                const uint32_t hh = __popc(ci);
                hits += hh;
                if (hh) atomicAdd(&cnt3[o], hh);
            }
            hits_total += hits;
            if (hits) atomicAdd(&ws.cnt[k], hits);
        }
#pragma unroll
        for (uint32_t g = 0; g < kPieceHigh / kPiece; ++g) {
            uint32_t d[kPiece];
#pragma unroll
            for (uint32_t i = 0; i < kPiece; ++i) d[i] = cm[g * kPiece + i];
            mc.add16(d);
        }
    }
    wave_lds_sync();
    if (ws.cnt[lane]) atomicAdd(&tpv[ws.beg[lane]], (unsigned long long)ws.cnt[lane]);
    wave_lds_sync();
    return hits_total;
}

// Per-vertex counts of the panels: the workgroup items of the panel region, from their own
// queue counter (every other item is left to k_count<true>).  The ranks above P are taken in
// windows of kPvWindow: per window, the table and the third-vertex counters cover its ranks,
// every segment is streamed whole, and entries outside the window clamp onto the zero word
// (one window for panels within kPvWindow ranks of the top, two for the rest of a region of
// up to 32,736 ranks).
__global__ __launch_bounds__(kThreads) void k_count_panel_pv(
    const uint32_t *__restrict__ row_ptr, const uint32_t *__restrict__ col,
    const uint32_t *__restrict__ cptr, const uint32_t *__restrict__ cbeg,
    const uint4 *__restrict__ er, const uint32_t *__restrict__ item_v_b,
    const uint32_t *__restrict__ item_off_b, const uint32_t *__restrict__ n_items_b_ptr,
    uint32_t *__restrict__ queue_c, unsigned long long *__restrict__ total,
    unsigned long long *__restrict__ tpv, uint32_t n1, const uint32_t *__restrict__ first_panel,
    uint32_t kitem_b,
    const uint16_t *__restrict__ hcol, uint32_t hbase, const int32_t *__restrict__ status) {
    __shared__ uint32_t s_mem[kLdsWords];
    __shared__ WaveScratch s_ws[kWaves];
    __shared__ unsigned long long s_mid[kPanel];
    __shared__ uint32_t s_item;
    if (*status) return;
    const uint32_t t = threadIdx.x, w = t / kWave, lane = lane_id();
    WaveScratch &ws = s_ws[w];
    const InEdgeSegs segs{cbeg, er};
    uint32_t *m = s_mem, *cnt3 = s_mem + kPvPanelWords;
    for (uint32_t i = t; i < kLdsWords; i += kThreads) s_mem[i] = 0;
    if (t < kPanel) s_mid[t] = 0;
    uint64_t acc = 0;
    MidCounters mc;
    mc.clear();
    const uint32_t n_items_b = *n_items_b_ptr;
    for (;;) {
        __syncthreads();
        if (t == 0) s_item = atomicAdd(queue_c, 1u);
        __syncthreads();
        uint32_t q = s_item;
        if (q >= n_items_b) break;
        q = n_items_b - 1 - q;
        const ItemRange it = item_range(q, kitem_b, n1, item_v_b, item_off_b, cptr, row_ptr);
        if (it.v < *first_panel) continue;  // left to k_count<true>
        const uint32_t P = it.v, np = min(kPanel, n1 - 1 - P);
        uint32_t cnt = 0, pieces = 0;
        // window of ranks [lo, lo + wn) above P (rank P itself is in no out-list of the panel)
        for (uint32_t lo = P; lo < n1 - 1; lo += kPvWindow) {
            const uint32_t wn = min(kPvWindow, n1 - 1 - lo);
            for (uint32_t j = w; j < np; j += kWaves)
                for (uint32_t i = row_ptr[P + j] + lane; i < row_ptr[P + j + 1]; i += kWave) {
                    const uint32_t o = col[i] - lo;
                    if (o < wn) atomicOr(&m[o], 1u << j);
                }
            __syncthreads();
            if (P >= hbase) {  // the suffixes are in hcol
                for (uint32_t eb = it.e0 + w * kWave; eb < it.e1; eb += kWaves * kWave) {
                    const SegRec r = eb + lane < it.e1 ? segs.rec(eb + lane)
                                                       : SegRec{0u, 0u, 0u, 0u, 0u};
                    cnt += run_panel_pv_high(r, hcol, m, cnt3, lo - hbase, wn, lo > P,
                                             lo + wn < n1 - 1, ws, mc, pieces, s_mid, tpv);
                }
            } else {
                for (uint32_t eb = it.e0 + w * kWave; eb < it.e1; eb += kWaves * kWave)
                    cnt += run_panel_pv(eb, it.e1, segs, col, m, cnt3, lo, wn - 1, ws, mc,
                                        pieces, s_mid, tpv);
            }
            __syncthreads();
            for (uint32_t j = w; j < np; j += kWaves)
                for (uint32_t i = row_ptr[P + j] + lane; i < row_ptr[P + j + 1]; i += kWave) {
                    const uint32_t o = col[i] - lo;
                    if (o < wn) m[o] = 0;
                }
            for (uint32_t i = t; i < wn; i += kThreads) {
                const uint32_t c3 = cnt3[i];
                if (c3) {
                    atomicAdd(&tpv[lo + i], (unsigned long long)c3);
                    cnt3[i] = 0;
                }
            }
            __syncthreads();
        }
        mc.flush(s_mid);
        acc += cnt;
        __syncthreads();
        if (t < np && s_mid[t]) {
            atomicAdd(&tpv[P + t], s_mid[t]);
            s_mid[t] = 0;
        }
    }
    acc = wave_sum_u64(acc);
    if (lane == 0 && acc) atomicAdd(total, (unsigned long long)acc);
}

// ------------------------------------------------------------------ the kernel

// c third-vertex credits to rank w: in LDS from rank hot0 on, 32 bits wide, whose carry goes to
// the count itself
__device__ __forceinline__ void credit_third(uint32_t w, uint32_t c, uint32_t hot0, uint32_t *hot,
                                             unsigned long long *__restrict__ tpv) {
    if (w >= hot0) {
        const uint32_t before = atomicAdd(&hot[w - hot0], c);
        if (before + c < before) atomicAdd(&tpv[w], 1ull << 32);
    } else {
        atomicAdd(&tpv[w], (unsigned long long)c);
    }
}

template <bool PV>
__global__ __launch_bounds__(kThreads) void k_count(
    const uint32_t *__restrict__ row_ptr, const uint32_t *__restrict__ col,
    const uint32_t *__restrict__ cptr, const uint32_t *__restrict__ cbeg,
    const uint4 *__restrict__ er, const uint32_t *__restrict__ item_v_a,
    const uint32_t *__restrict__ item_off_a, const uint32_t *__restrict__ n_items_a_ptr,
    const uint32_t *__restrict__ item_v_b, const uint32_t *__restrict__ item_off_b,
    const uint32_t *__restrict__ n_items_b_ptr, uint32_t *__restrict__ queue_a,
    uint32_t *__restrict__ queue_b, unsigned long long *__restrict__ total,
    unsigned long long *__restrict__ tpv, uint32_t n1, const uint32_t *__restrict__ first_panel,
    uint32_t wave_bits,
    uint32_t block_bits, uint32_t block_list, uint32_t kitem_a, uint32_t kitem_b,
    const uint16_t *__restrict__ hcol, const uint32_t *__restrict__ hrow, uint32_t hbase,
    const unsigned long long *__restrict__ light_total, const int32_t *__restrict__ status) {
    // 8 KiB aligned: a wave slice's base has zero low bits, so bitmap addresses OR it in
    __shared__ __attribute__((aligned(kSliceWords * 4))) uint32_t s_mem[kLdsWords];
    __shared__ WaveScratch s_ws[kWaves];
    __shared__ uint32_t s_item;
    __shared__ uint32_t s_hot[PV ? kHotRanks : 1];
    if (*status) return;
    const uint32_t t = threadIdx.x, w = t / kWave, lane = lane_id();
    WaveScratch &ws = s_ws[w];
    const InEdgeSegs segs{cbeg, er};
    for (uint32_t i = t; i < kLdsWords; i += kThreads) s_mem[i] = 0;
    const uint32_t hot0 = n1 - 1 > kHotRanks ? n1 - 1 - kHotRanks : 0u;
    if (PV && t < kHotRanks) s_hot[t] = 0;
    uint64_t acc = 0;
    if (blockIdx.x == 0 && t < kLightTotals) acc = light_total[t * kLightTotalStep];

    const uint32_t p0 = *first_panel;
    // phase 1: workgroup items
    const uint32_t n_items_b = *n_items_b_ptr;
    for (;;) {
        __syncthreads();
        if (t == 0) s_item = atomicAdd(queue_b, 1u);
        __syncthreads();
        uint32_t q = s_item;
        if (q >= n_items_b) break;
        q = n_items_b - 1 - q;
        const ItemRange it = item_range(q, kitem_b, n1, item_v_b, item_off_b, cptr, row_ptr);
        const uint32_t first = it.e0 + w * kWave, step = kWaves * kWave;
        if (it.v >= p0) {  // a panel of middle vertices P = it.v, ...
            const uint32_t P = it.v, np = min(kPanel, n1 - 1 - P);
            if (!PV) {
                for (uint32_t j = w; j < np; j += kWaves)
                    for (uint32_t i = row_ptr[P + j] + lane; i < row_ptr[P + j + 1]; i += kWave)
                        atomicOr(&s_mem[col[i] - P], 1u << j);
                __syncthreads();
                uint32_t cnt = 0;
                if (P >= hbase) {  // the suffixes are in hcol
                    const PanelHighProbe probe{s_mem, P - hbase};
                    cnt += stream_t(first, it.e1, step, segs, col, hcol, hbase, probe, ws);
                } else {  // no high region: 32-bit entries
                    const PanelProbe probe{s_mem, P, n1 - 2 - P};
                    for (uint32_t eb = first; eb < it.e1; eb += step)
                        cnt += run_batch<false>(eb, it.e1, segs, col, probe, ws, nullptr, tpv);
                }
                acc += cnt;
                __syncthreads();
                for (uint32_t j = w; j < np; j += kWaves)
                    for (uint32_t i = row_ptr[P + j] + lane; i < row_ptr[P + j + 1]; i += kWave)
                        s_mem[col[i] - P] = 0;
            }
            continue;
        }
        const uint32_t lo = col[it.r0];
        const uint32_t span = col[it.r0 + it.d - 1] - lo;
        // 0 = bitmap, 1 = LDS list, 2 = global list (block_bits <= kBlockBits, block_list <=
        // kBlockList, or kBlockListPV for per-vertex counts)
        const int mode = (!PV && span < block_bits) ? 0 : (it.d <= block_list) ? 1 : 2;
        if (mode == 0) {
            for (uint32_t i = t; i < it.d; i += kThreads) {
                const uint32_t o = col[it.r0 + i] - lo;
                atomicOr(&s_mem[o >> 5], 1u << (o & 31u));
            }
        } else if (mode == 1) {
            for (uint32_t i = t; i < it.d; i += kThreads) s_mem[i] = col[it.r0 + i];
        }
        __syncthreads();
        uint32_t cnt = 0;
        if (mode == 0) {
            if constexpr (!PV) {
                const BitmapProbe probe{s_mem, lo, span};
                cnt += stream_t(first, it.e1, step, segs, col, hcol, hbase, probe, ws);
            }
        } else if (mode == 1) {
            const LdsListProbe probe{lds_addr(s_mem), it.d};
            uint32_t *tc = PV ? s_mem + kBlockListPV : nullptr;
            if constexpr (PV) {
                for (uint32_t eb = first; eb < it.e1; eb += step)
                    cnt += run_batch<true>(eb, it.e1, segs, col, probe, ws, tc, tpv);
            } else {
                cnt += stream_t(first, it.e1, step, segs, col, hcol, hbase, probe, ws);
            }
        } else {
            const ListProbe probe{col + it.r0, it.d};
            if constexpr (PV) {
                for (uint32_t eb = first; eb < it.e1; eb += step)
                    cnt += run_batch<true>(eb, it.e1, segs, col, probe, ws, nullptr, tpv);
            } else {
                cnt += stream_t(first, it.e1, step, segs, col, hcol, hbase, probe, ws);
            }
        }
        if (PV) {
            uint64_t wave_hits = wave_sum_u64(cnt);
            if (lane == 0 && wave_hits) atomicAdd(&tpv[it.v], (unsigned long long)wave_hits);
        }
        acc += cnt;
        __syncthreads();
        if (mode == 0) {
            for (uint32_t i = t; i < it.d; i += kThreads) s_mem[(col[it.r0 + i] - lo) >> 5] = 0;
        } else if (mode == 1) {
            for (uint32_t i = t; i < it.d; i += kThreads) {
                s_mem[i] = 0;
                if (PV) {
                    uint32_t c = s_mem[kBlockListPV + i];
                    if (c) {
                        credit_third(col[it.r0 + i], c, hot0, s_hot, tpv);
                        s_mem[kBlockListPV + i] = 0;
                    }
                }
            }
        }
    }
    __syncthreads();

    // phase 2: wave items, each wave in its own LDS slice
    uint32_t *mem = s_mem + w * kSliceWords;
    // the high-region bitmap ORs the slice's address into its word offsets (requested by the
    // alignment of s_mem; otherwise the span bitmap takes its items)
    const bool slices_aligned = (lds_addr(s_mem) & (kSliceWords * 4 - 1)) == 0;
    const uint32_t n_items_a = *n_items_a_ptr;
    WaveQueue wq{kClaimWave};
    for (uint32_t q; wq.pop(queue_a, n_items_a, q);) {
        q = n_items_a - 1 - q;
        const ItemRange it = item_range(q, kitem_a, n1, item_v_a, item_off_a, cptr, row_ptr);
        uint32_t cnt = 0;
        if (!PV) {
            const uint32_t lo = col[it.r0];
            const uint32_t span = col[it.r0 + it.d - 1] - lo;
            if (span < wave_bits && it.v >= hbase && slices_aligned) {
                // bitmap over the whole high region (N+(v) lies in it; the slice holds 2^16
                // bits); every in-edge suffix is high
                for (uint32_t i = lane; i < it.d; i += kWave) {
                    const uint32_t x = col[it.r0 + i] - hbase;
                    atomicOr(&mem[x >> 5], 1u << (x & 31u));
                }
                wave_lds_sync();
                const HighBitmapProbe probe{lds_addr(mem)};
                cnt += stream_t(it.e0, it.e1, kWave, segs, col, hcol, hbase, probe, ws);
                for (uint32_t i = lane; i < it.d; i += kWave)
                    mem[(col[it.r0 + i] - hbase) >> 5] = 0;
            } else if (span < wave_bits) {  // bitmap over the span
                for (uint32_t i = lane; i < it.d; i += kWave) {
                    const uint32_t o = col[it.r0 + i] - lo;
                    atomicOr(&mem[o >> 5], 1u << (o & 31u));
                }
                wave_lds_sync();
                const BitmapProbe probe{mem, lo, span};
                cnt += stream_t(it.e0, it.e1, kWave, segs, col, hcol, hbase, probe, ws);
                for (uint32_t i = lane; i < it.d; i += kWave)
                    mem[(col[it.r0 + i] - lo) >> 5] = 0;
            } else if (hbase + 1 < n1 && slices_aligned) {
                // a wide span (a list of at most wave_list_max <= kSliceWords entries, see
                // k_items): the suffixes' entries below hbase against N+(v)'s entries below
                // hbase as a sorted list, their entries >= hbase against N+(v)'s in the
                // high-region bitmap; with the list in the slice too, which the bitmap fills, one
                // after the other (no pass for a part N+(v) lacks)
                const uint32_t hr = hrow[it.v];
                const uint32_t dlo = hr == ~0u ? it.d : hr - it.r0;
                // up to kWave entries below hbase fit the wave's scratch: one pass, which gathers
                // the records once (missed lines are what these items are bound by).  R-MAT 23,
                // where 93 percent of the 561,000 wide lists are that short: 26.37 ms a step with
                // two passes for all, 25.91 with one for these
                const bool both = dlo > 0 && dlo <= kWave && dlo < it.d;
                if (both) {
                    if (lane < dlo) ws.cnt[lane] = col[it.r0 + lane];
                } else if (dlo > 0) {
                    for (uint32_t i = lane; i < dlo; i += kWave) mem[i] = col[it.r0 + i];
                    wave_lds_sync();
                    const LdsListProbe lp{lds_addr(mem), dlo};
                    cnt += stream_t<1>(it.e0, it.e1, kWave, segs, col, hcol, hbase, lp, ws);
                    for (uint32_t i = lane; i < dlo; i += kWave) mem[i] = 0;
                    wave_lds_sync();
                }
                for (uint32_t i = dlo + lane; i < it.d; i += kWave) {
                    const uint32_t x = col[it.r0 + i] - hbase;
                    atomicOr(&mem[x >> 5], 1u << (x & 31u));
                }
                wave_lds_sync();
                const HighMaskedProbe probe{HighBitmapProbe{lds_addr(mem)}};
                if (both) {
                    const LowHighProbe lh{LdsListProbe{lds_addr(ws.cnt), dlo}, probe};
                    cnt += stream_t(it.e0, it.e1, kWave, segs, col, hcol, hbase, lh, ws);
                } else if (dlo < it.d) {
                    cnt += stream_t<2>(it.e0, it.e1, kWave, segs, col, hcol, hbase, probe, ws);
                }
                for (uint32_t i = dlo + lane; i < it.d; i += kWave)
                    mem[(col[it.r0 + i] - hbase) >> 5] = 0;
            } else {  // a wide span, but a list that fits the slice (see k_items)
                for (uint32_t i = lane; i < it.d; i += kWave) mem[i] = col[it.r0 + i];
                wave_lds_sync();
                const LdsListProbe probe{lds_addr(mem), it.d};
                cnt += stream_t(it.e0, it.e1, kWave, segs, col, hcol, hbase, probe, ws);
                for (uint32_t i = lane; i < it.d; i += kWave) mem[i] = 0;
            }
            wave_lds_sync();
        } else {
            // with the filter up to kFilterList entries, else list and counters in half a slice
            // each; the counters and the filter are zero between items
            const bool filtered = it.d <= kFilterList;
            uint32_t *list = mem, *tc = mem + (filtered ? kFilterList : kWaveListPV);
            uint32_t *filter = mem + 2 * kFilterList;
            for (uint32_t i = lane; i < it.d; i += kWave) {
                const uint32_t x = col[it.r0 + i];
                list[i] = x;
                if (filtered)
                    atomicOr(&filter[(x & (kFilterBits - 1u)) >> 5], 1u << (x & 31u));
                else
                    tc[i] = 0;  // (the hit queue's words)
            }
            wave_lds_sync();
            if (filtered) {
                for (uint32_t eb = it.e0; eb < it.e1; eb += kWave)
                    cnt += run_filter_pv(eb, it.e1, segs, col, mem, it.d, ws, tpv);
            } else {
                const LdsListProbe probe{lds_addr(list), it.d};
                for (uint32_t eb = it.e0; eb < it.e1; eb += kWave)
                    cnt += run_batch<true>(eb, it.e1, segs, col, probe, ws, tc, tpv);
            }
            for (uint32_t i = lane; i < it.d; i += kWave) {
                const uint32_t x = list[i], c = tc[i];
                if (filtered)
                    filter[(x & (kFilterBits - 1u)) >> 5] = 0;
                else
                    list[i] = 0;  // (the counters of filtered items)
                if (c) {
                    credit_third(x, c, hot0, s_hot, tpv);
                    tc[i] = 0;
                }
            }
            uint64_t item_hits = wave_sum_u64(cnt);
            if (lane == 0 && item_hits) atomicAdd(&tpv[it.v], (unsigned long long)item_hits);
            wave_lds_sync();
        }
        acc += cnt;
    }
    acc = wave_sum_u64(acc);
    if (lane == 0 && acc) atomicAdd(total, (unsigned long long)acc);
    if constexpr (PV) {
        __syncthreads();
        if (t < kHotRanks && s_hot[t]) atomicAdd(&tpv[hot0 + t], (unsigned long long)s_hot[t]);
    }
}

// ------------------------------------------------------------------ batched kernel

// Batched counting over a disjoint union of small graphs in id space (their oriented lists
// keep the input's id order, no relabelling).  Every triangle is found once, from its first
// vertex u in the order of Section 2.2: for every out-neighbour v of u, the common elements of
// N+(u) and N+(v).
//   heavy items (k_count_u; u with d+(u) > light_max): (u, chunk of up to kitem out-neighbours
//     of u); N+(u) is staged in the wave's LDS slice (bitmap over its id span, or a sorted list)
//     and the whole list N+(v) of every out-neighbour v streams through it.  Hits go to the
//     graph of u; per-vertex counts credit u (per item), v (per segment) and w (LDS counters by
//     list position).
//   light rows (k_count_light): a wave takes 2^vshift consecutive vertices, stages their light
//     rows (whole rows, up to `window` entries at a time) in LDS, one edge u -> v per lane.

template <bool PV>
__global__ __launch_bounds__(kThreads) void k_count_u(const BatchKernelArgs a) {
    __shared__ uint32_t s_mem[kLdsWords];
    __shared__ WaveScratch s_ws[kWaves];
    const uint32_t n_items = *a.n_items, kitem = a.kitem;
    if (n_items == 0) return;
    const uint32_t t = threadIdx.x, w = t / kWave, lane = lane_id();
    WaveScratch &ws = s_ws[w];
    uint32_t *mem = s_mem + w * kSliceWords;
    for (uint32_t i = t; i < kLdsWords; i += kThreads) s_mem[i] = 0;
    __syncthreads();
    const uint32_t *__restrict__ fcol = a.fcol;
    unsigned long long *totals = *a.totals_pp;
    unsigned long long *tpv = PV ? *a.tpv_pp : nullptr;
    const OutEdgeSegs segs{a.frow, fcol};
    // few items: one per claim, so that they spread over the waves (64 per claim put the hub
    // rows of a few small graphs on two or three waves)
    const uint32_t share = n_items / (gridDim.x * kWaves * 4);
    WaveQueue wq{min(max(share, 1u), kClaimBatched)};
    for (uint32_t q; wq.pop(a.queue, n_items, q);) {
        const uint2 item = a.items[q];
        const uint32_t u = item.x, e0 = item.y;
        const uint2 ru = a.frow[u];
        const uint32_t r0 = ru.x, d = ru.y - r0;
        const uint32_t e1 = min(e0 + kitem, r0 + d);
        uint32_t lo = ~0u, hi = 0;  // the id span of N+(u) (rows of invalid graphs may be
        for (uint32_t i = lane; i < d; i += kWave) {  // unsorted, so take min and max)
            const uint32_t x = fcol[r0 + i];
            lo = min(lo, x);
            hi = max(hi, x);
        }
        for (int o = kWave / 2; o >= 1; o >>= 1) {
            lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, kWave));
            hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, kWave));
        }
        const uint32_t span = hi - lo;
        // 0 = bitmap in the slice, 1 = sorted list in the slice, 2 = sorted list in memory
        // (a.wave_bits <= kWaveBits; a.wave_list <= kSliceWords, or kWaveListPV per vertex)
        const int mode = (!PV && span < a.wave_bits) ? 0 : (d <= a.wave_list) ? 1 : 2;
        uint32_t cnt = 0;
        if (mode == 0) {
            for (uint32_t i = lane; i < d; i += kWave) {
                const uint32_t o = fcol[r0 + i] - lo;
                atomicOr(&mem[o >> 5], 1u << (o & 31u));
            }
            wave_lds_sync();
            if constexpr (!PV) {
                const BitmapProbe probe{mem, lo, span};
                for (uint32_t eb = e0; eb < e1; eb += kWave)
                    cnt += run_batch<false>(eb, e1, segs, fcol, probe, ws, nullptr, tpv);
            }
            for (uint32_t i = lane; i < d; i += kWave) mem[(fcol[r0 + i] - lo) >> 5] = 0;
        } else if (mode == 1) {
            uint32_t *list = mem, *tc = PV ? mem + kWaveListPV : nullptr;
            for (uint32_t i = lane; i < d; i += kWave) list[i] = fcol[r0 + i];
            wave_lds_sync();
            const LdsListProbe probe{lds_addr(list), d};
            for (uint32_t eb = e0; eb < e1; eb += kWave)
                cnt += run_batch<PV>(eb, e1, segs, fcol, probe, ws, tc, tpv);
            for (uint32_t i = lane; i < d; i += kWave) {
                list[i] = 0;
                if (PV && tc[i]) {
                    atomicAdd(&tpv[fcol[r0 + i]], (unsigned long long)tc[i]);
                    tc[i] = 0;
                }
            }
        } else {
            const ListProbe probe{fcol + r0, d};
            for (uint32_t eb = e0; eb < e1; eb += kWave)
                cnt += run_batch<PV>(eb, e1, segs, fcol, probe, ws, nullptr, tpv);
        }
        wave_lds_sync();
        const uint64_t item_hits = wave_sum_u64(cnt);
        if (lane == 0 && item_hits) {
            atomicAdd(&totals[a.gid[u]], (unsigned long long)item_hits);
            if (PV) atomicAdd(&tpv[u], (unsigned long long)item_hits);
        }
    }
}

// ------------------------------------------------------------------ light rows

// four entries from a 4-byte aligned position
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// A piece of up to kLightPiece entries of N+(v) (wv, the first `cnt` of them valid) against the
// staged list at LDS byte address lb (d >= 1 ascending entries): bit kLightPiece - 1 - i of the
// result is set when wv[i] is in the list, and at[i] is the byte address of the last list entry
// <= wv[i] (lb when none is).  The piece's binary searches advance in lockstep, three vector
// operations and one LDS read per step; lanes whose range is down to one entry stay put.
__device__ __forceinline__ uint32_t light_piece(const uint32_t (&wv)[kLightPiece], uint32_t cnt,
                                                uint32_t lb, uint32_t d,
                                                uint32_t (&at)[kLightPiece]) {
#pragma unroll
    for (uint32_t i = 0; i < kLightPiece; ++i) at[i] = lb;
    uint32_t left = cnt ? d * 4u : 4u;  // bytes
    // the longest range of the wave sets the steps (a scalar loop)
    uint32_t most = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_max(left), kWave - 1);
    for (; most > 4u; most -= (most >> 1) & ~3u) {
        const uint32_t half = (left >> 1) & ~3u;
#pragma unroll
        for (uint32_t i = 0; i < kLightPiece; ++i) {
            const uint32_t mid = at[i] + half;
            at[i] = lds_word(mid) <= wv[i] ? mid : at[i];
        }
        left -= half;
    }
    uint32_t packed = 0;
#pragma unroll
    for (uint32_t i = 0; i < kLightPiece; ++i)
        packed = packed + packed + (lds_word(at[i]) == wv[i] ? 1u : 0u);
    return packed & ~((1u << (kLightPiece - min(cnt, kLightPiece))) - 1u);
}

__device__ __forceinline__ void load_light_piece(const uint32_t *__restrict__ fcol, uint32_t at,
                                                 uint32_t (&wv)[kLightPiece]) {
    const u32x4_a4 *p = reinterpret_cast<const u32x4_a4 *>(fcol + at);
#pragma unroll
    for (uint32_t j = 0; j < kLightPiece / 4; ++j) {
        const u32x4_a4 x = p[j];
        wv[4 * j] = x[0];
        wv[4 * j + 1] = x[1];
        wv[4 * j + 2] = x[2];
        wv[4 * j + 3] = x[3];
    }
}

// Bound by its vector instructions on 4096 graphs of 3300 vertices (80% of the issue slots), not
// by memory: so the first piece of every list runs on the lane that owns the edge, with nothing
// passed between lanes; only the further pieces of longer lists are dealt out, in full rounds
// of 64 (a part of a round waits for the next 64 edges' pieces).  A wave's hits need no
// attribution to edges for totals: rows of one graph are taken together and summed once.  An XCD
// takes stretches of consecutive rows (xcd_stretch_tile), since a graph's lists are read by its
// neighbours: dealt round-robin, every XCD's L2 fetched every graph (1.2e8 lines missed instead of
// 4.4e7).  The batch above: 1.74 ms, 3.0 ms when a persistent kernel took chunks of edges.
//
// Per-vertex counts: a triangle u, v, w (v and w in N+(u)) is found from the edge u -> v with w
// in N+(v), and credits the window's counters of the entries v and w of row u.  They are added
// to T once per entry (one memory atomic per edge that closes triangles, where crediting u, v
// and w by themselves took one per triangle and two per edge), and T(u) is half of their sum:
// 300 graphs of 9.0e6 edges took 1630 us, bound by those atomics, and take 340 us.
template <bool PV>
__global__ __launch_bounds__(kLightThreads, 8) void k_count_light(const BatchKernelArgs a,
                                                               uint32_t vshift) {
    extern __shared__ uint32_t s_dyn[];
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t per = a.window + a.window / 4 + kWave + (PV ? a.window : 0u);
    uint32_t *mark = s_dyn + w * per;                           // kWave words
    uint32_t *list = mark + kWave;                              // window entries
    uint8_t *own = (uint8_t *)(list + a.window);                // the row of every entry
    uint32_t *cnt3 = list + a.window + a.window / 4;            // PV: counters of the entries
    const uint32_t N = *a.n;
    const uint32_t x0 = (xcd_stretch_tile(blockIdx.x, gridDim.x) * kLightWaves + w) << vshift;
    if (x0 >= N) return;
    const uint32_t *__restrict__ fcol = a.fcol;
    const uint32_t x = x0 + lane;
    uint2 row = make_uint2(0u, 0u);
    uint32_t g = ~0u;
    if ((lane >> vshift) == 0 && x < N) {
        row = a.frow[x];
        g = a.gid[x];
    }
    uint32_t len = row.y - row.x;
    if (len < 2 || len > a.light_max) len = 0;
    unsigned long long *totals = *a.totals_pp;
    unsigned long long *tpv = PV ? *a.tpv_pp : nullptr;
    const int64_t *vtx_off = *a.vtx_off_pp;
    uint64_t part = 0;  // lanes 0 and 1: this wave's parts of graphs that span waves
    mark[lane] = 0;
    uint32_t round = 0;
    const uint32_t list_b = lds_addr(list);
    for (uint64_t todo = __ballot(len > 0); todo;) {
        // the rows of one graph (nearly always all of the wave's)
        const uint32_t gc = (uint32_t)__builtin_amdgcn_readlane((int)g, __ffsll((long long)todo) - 1);
        const bool mine = len > 0 && g == gc;
        todo &= ~__ballot(mine);
        const uint32_t mlen = mine ? len : 0u;
        const uint32_t incl = wave_incl_scan(mlen);
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        uint32_t hits = 0;
        for (uint32_t w0 = 0; w0 < all;) {  // windows of whole rows (window >= light_max)
            const bool in = mine && incl - mlen >= w0 && incl <= w0 + a.window;
            const uint64_t in_mask = __ballot(in);
            const uint32_t w1 = (uint32_t)__builtin_amdgcn_readlane(
                (int)incl, 63 - __builtin_clzll(in_mask));
            const uint32_t n = w1 - w0;
            const uint32_t off = incl - mlen - w0;
            // stage the rows, and the row of every entry
            uint32_t carry = 0;
            const uint32_t delta = row.x - off;
            for (uint32_t i0 = 0; i0 < n; i0 += kWave) {
                const uint32_t k = round_owner(mark, off, in, i0, ++round, carry) - 1u;
                const uint32_t dk = wave_bcast_from(delta, k);
                const uint32_t i = i0 + lane;
                if (i < n) {
                    list[i] = fcol[dk + i];
                    own[i] = (uint8_t)k;
                    if (PV) cnt3[i] = 0;
                }
            }
            wave_lds_sync();
            const uint32_t ol = in ? (off | (mlen << 16)) : 0u;
            // pieces waiting for a full round: lane l < waiting holds one (its start in fcol,
            // entries, staged list and edge)
            uint32_t waiting = 0, pb = 0, pc = 0, pr = 0, pe = 0;
            uint32_t wv[kLightPiece], at[kLightPiece];
            auto credit = [&](uint32_t packed, uint32_t edge) {
                hits += (uint32_t)__popc(packed);
                if (PV && packed) {
                    atomicAdd(&cnt3[edge], (uint32_t)__popc(packed));
#pragma unroll
                    for (uint32_t j = 0; j < kLightPiece; ++j)
                        if ((packed >> (kLightPiece - 1 - j)) & 1u)
                            atomicAdd(&cnt3[(at[j] - list_b) >> 2], 1u);
                }
            };
            auto run_waiting = [&]() {
                if (pc) load_light_piece(fcol, pb, wv);
                credit(light_piece(wv, pc, list_b + (pr & 0xFFFFu) * 4u, pr >> 16, at), pe);
            };
            for (uint32_t i0 = 0; i0 < n; i0 += kWave) {
                const uint32_t i = i0 + lane;
                const bool valid = i < n;
                const uint32_t rk = wave_bcast_from(ol, valid ? (uint32_t)own[i] : 0u);
                uint2 rv = make_uint2(0u, 0u);
                if (valid) rv = a.frow[list[i]];
                const uint32_t c = rv.y - rv.x;
                if (c) load_light_piece(fcol, rv.x, wv);
                credit(light_piece(wv, c, list_b + (rk & 0xFFFFu) * 4u, rk >> 16, at), i);
                // further pieces of longer lists, after the waiting ones; the last, partly
                // filled round waits
                const uint32_t p = c > kLightPiece ? (c - 1) / kLightPiece : 0u;
                if (__ballot(p != 0) == 0) continue;
                const uint32_t pincl = wave_incl_scan(p);
                const uint32_t my_off = waiting + pincl - p;
                const uint32_t Q =
                    waiting + (uint32_t)__builtin_amdgcn_readlane((int)pincl, kWave - 1);
                uint32_t pcarry = 0;
                for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
                    const uint32_t k = round_owner(mark, my_off, p, q0, ++round, pcarry) - 1u;
                    const uint32_t q = q0 + lane - wave_bcast_from(my_off, k);
                    const uint32_t b = wave_bcast_from(rv.x, k) + (q + 1u) * kLightPiece;
                    const uint32_t en = wave_bcast_from(rv.y, k);
                    const uint32_t rq = wave_bcast_from(rk, k);
                    if (q0 + lane >= waiting) {
                        pb = b;
                        pc = q0 + lane < Q ? en - b : 0u;
                        pr = rq;
                        pe = i0 + k;
                    }
                    waiting = Q - q0;  // (from this round on)
                    if (waiting < kWave) break;
                    run_waiting();
                    waiting = 0;
                }
            }
            if (waiting) run_waiting();
            wave_lds_sync();
            if (PV) {
                for (uint32_t i = lane; i < n; i += kWave)
                    if (cnt3[i]) atomicAdd(&tpv[list[i]], (unsigned long long)cnt3[i]);
                uint32_t sum = 0;
                if (in)
                    for (uint32_t j = 0; j < mlen; ++j) sum += cnt3[off + j];
                if (sum) atomicAdd(&tpv[x], (unsigned long long)(sum / 2));
                wave_lds_sync();
            }
            w0 = w1;
        }
        const uint64_t sum = wave_sum_u64(hits);
        const uint32_t span = graph_span(vtx_off, gc, x0, vshift);
        if (span == kSpanWhole) {
            if (lane == 0 && sum) totals[gc] += sum;  // (no other wave adds to it meanwhile)
        } else if (lane == span) {
            part = sum;
        }
    }
    if (lane < 2) a.wtotal[2 * (x0 >> vshift) + lane] = part;
}

// ------------------------------------------------------------------ light middle vertices
//
// The lists of vertices v below the first panel with few in-edges and a short N+(v) (kLightList):
// a wave takes up to 16 consecutive lists (at R-MAT 20 the densest waves of 64 lists ran on for 100
// us after the others, 1960 against 1913 us a count), stages their N+(v) in LDS (whole lists, a
// window at a time) and takes their in-edges u -> v one per lane, whatever list they belong to:
// the suffix of N+(u) after v (short as well: u comes before v in the order of degrees) is looked
// up in N+(v) by binary search, its first piece on the edge's own lane, further pieces in full
// rounds.
//
// Per-vertex counts: a hit credits an LDS counter of N+(v)'s entry (added to T(w) once per entry,
// and their sum to T(v)) and T(u) once per piece.  The highest ranks' T(w) go through LDS counters of
// the workgroup: where a few hubs are in every list, the atomics on them are most of the work (a
// ring of 200,000 vertices joined to three hubs: 2758 us a count without these sums, 819 with).
template <bool PV>
__global__ __launch_bounds__(kLightThreads) void k_count_light_lists(
    const uint32_t *__restrict__ row_ptr, const uint32_t *__restrict__ col,
    const uint32_t *__restrict__ cptr, const uint32_t *__restrict__ cbeg,
    const uint4 *__restrict__ er, uint32_t lists, uint32_t n1,
    const uint32_t *__restrict__ first_panel, uint32_t light, uint32_t lshift,
    unsigned long long *__restrict__ light_total, unsigned long long *__restrict__ tpv,
    const int32_t *__restrict__ status) {
    __shared__ uint32_t s_mark[kLightWaves][kWave];
    __shared__ uint32_t s_list[kLightWaves][kLightListWindow];
    __shared__ uint32_t s_cnt[kLightWaves][PV ? kLightListWindow : 1];
    __shared__ uint32_t s_hot[PV ? kHotRanks : 1];
    if (*status) return;
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t hot0 = n1 - 1 > kHotRanks ? n1 - 1 - kHotRanks : 0u;
    if constexpr (PV) {
        for (uint32_t i = threadIdx.x; i < kHotRanks; i += kLightThreads) s_hot[i] = 0;
        __syncthreads();
    }
    const uint32_t tile = xcd_stretch_tile(blockIdx.x, gridDim.x);
    const uint32_t c = (lane >> lshift) == 0 ? ((tile * kLightWaves + w) << lshift) + lane : lists;
    uint32_t *mark = s_mark[w], *list = s_list[w], *cnt3 = s_cnt[w];
    uint32_t cb = 0, in_edges = 0, r0 = 0, d = 0, v = 0;
    if (c < lists) {
        v = c < n1 ? c : c % n1;
        if (v < *first_panel) {
            cb = cptr[c];
            in_edges = cptr[c + 1] - cb;
            r0 = row_ptr[v];
            d = row_ptr[v + 1] - r0;
        }
    }
    if (in_edges > light || d > light || in_edges == 0) d = 0;
    mark[lane] = 0;
    uint32_t round = 0, hits = 0;
    const uint32_t list_b = lds_addr(list);
    const uint32_t incl = wave_incl_scan(d);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    for (uint32_t w0 = 0; w0 < all;) {  // windows of whole lists
        const bool in = d > 0 && incl - d >= w0 && incl <= w0 + kLightListWindow;
        const uint64_t in_mask = __ballot(in);
        const uint32_t w1 =
            (uint32_t)__builtin_amdgcn_readlane((int)incl, 63 - __builtin_clzll(in_mask));
        const uint32_t n = w1 - w0, off = incl - d - w0;
        const uint32_t delta = r0 - off;
        uint32_t carry = 0;
        for (uint32_t i0 = 0; i0 < n; i0 += kWave) {
            const uint32_t k = round_owner(mark, off, in, i0, ++round, carry) - 1u;
            const uint32_t dk = wave_bcast_from(delta, k);
            const uint32_t i = i0 + lane;
            if (i < n) {
                list[i] = col[dk + i];
                if (PV) cnt3[i] = 0;
            }
        }
        wave_lds_sync();
        const uint32_t ol = off | (d << 16);
        const uint32_t ne = in ? in_edges : 0u;
        const uint32_t eincl = wave_incl_scan(ne), eoff = eincl - ne;
        const uint32_t edges = (uint32_t)__builtin_amdgcn_readlane((int)eincl, kWave - 1);
        const uint32_t edelta = cb - eoff;
        // pieces waiting for a full round: lane l < waiting holds one
        uint32_t waiting = 0, pb = 0, pc = 0, pr = 0, pu = 0, ecarry = 0;
        uint32_t wv[kLightPiece], at[kLightPiece];
#pragma unroll
        for (uint32_t j = 0; j < kLightPiece; ++j) wv[j] = 0;
        auto credit = [&](uint32_t packed, uint32_t u) {
            hits += (uint32_t)__popc(packed);
            if (PV && packed) {
                atomicAdd(&tpv[u], (unsigned long long)__popc(packed));
#pragma unroll
                for (uint32_t j = 0; j < kLightPiece; ++j)
                    if ((packed >> (kLightPiece - 1 - j)) & 1u)
                        atomicAdd(&cnt3[(at[j] - list_b) >> 2], 1u);
            }
        };
        auto run_waiting = [&]() {
            if (pc) load_light_piece(col, pb, wv);
            credit(light_piece(wv, pc, list_b + (pr & 0xFFFFu) * 4u, pr >> 16, at), pu);
        };
        for (uint32_t i0 = 0; i0 < edges; i0 += kWave) {
            const uint32_t k = round_owner(mark, eoff, ne, i0, ++round, ecarry) - 1u;
            const uint32_t j = wave_bcast_from(edelta, k) + i0 + lane;
            const uint32_t rk = wave_bcast_from(ol, k);
            uint32_t b = 0, en = 0, u = 0;
            if (i0 + lane < edges) {
                b = cbeg[j];
                const uint4 r = er[b - 1];
                en = r.x;
                u = r.w;
            }
            const uint32_t len = en - b;
            if (len) load_light_piece(col, b, wv);
            credit(light_piece(wv, len, list_b + (rk & 0xFFFFu) * 4u, rk >> 16, at), u);
            const uint32_t p = len > kLightPiece ? (len - 1) / kLightPiece : 0u;
            if (__ballot(p != 0) == 0) continue;
            const uint32_t pincl = wave_incl_scan(p);
            const uint32_t my_off = waiting + pincl - p;
            const uint32_t Q =
                waiting + (uint32_t)__builtin_amdgcn_readlane((int)pincl, kWave - 1);
            uint32_t pcarry = 0;
            for (uint32_t q0 = 0; q0 < Q; q0 += kWave) {
                const uint32_t kq = round_owner(mark, my_off, p, q0, ++round, pcarry) - 1u;
                const uint32_t q = q0 + lane - wave_bcast_from(my_off, kq);
                const uint32_t qb = wave_bcast_from(b, kq) + (q + 1u) * kLightPiece;
                const uint32_t qe = wave_bcast_from(en, kq);
                const uint32_t rq = wave_bcast_from(rk, kq);
                const uint32_t uq = PV ? wave_bcast_from(u, kq) : 0u;
                if (q0 + lane >= waiting) {
                    pb = qb;
                    pc = q0 + lane < Q ? qe - qb : 0u;
                    pr = rq;
                    pu = uq;
                }
                waiting = Q - q0;  // (from this round on)
                if (waiting < kWave) break;
                run_waiting();
                waiting = 0;
            }
        }
        if (waiting) run_waiting();
        wave_lds_sync();
        if (PV) {
            for (uint32_t i = lane; i < n; i += kWave)
                if (cnt3[i]) credit_third(list[i], cnt3[i], hot0, s_hot, tpv);
            uint32_t sum = 0;
            if (in)
                for (uint32_t j = 0; j < d; ++j) sum += cnt3[off + j];
            if (sum) atomicAdd(&tpv[v], (unsigned long long)sum);
            wave_lds_sync();
        }
        w0 = w1;
    }
    const uint64_t sum = wave_sum_u64(hits);
    // (one counter for all waves would queue them, 11 ns each)
    if (lane == 0 && sum)
        atomicAdd(&light_total[tile % kLightTotals * kLightTotalStep], (unsigned long long)sum);
    if constexpr (PV) {
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < kHotRanks; i += kLightThreads)
            if (s_hot[i]) atomicAdd(&tpv[hot0 + i], (unsigned long long)s_hot[i]);
    }
}

uint32_t count_light_window(uint32_t chunk, uint32_t light_max) {
    const uint32_t w = chunk > light_max ? chunk : light_max;
    return (w + 63u) & ~63u;
}

hipError_t launch_count_u(const BatchKernelArgs &a, bool per_vertex, uint32_t heavy_wgs,
                          uint32_t ncap, uint32_t vshift, hipStream_t s) {
    const dim3 lg(ceil_div(ceil_div(ncap > 0 ? ncap : 1, 1ull << vshift), kLightWaves));
    const size_t lds = (size_t)kLightWaves * 4 *
                       (a.window + a.window / 4 + kWave + (per_vertex ? a.window : 0));
    if (per_vertex) {
        hipLaunchKernelGGL(k_count_u<true>, dim3(heavy_wgs), dim3(kThreads), 0, s, a);
        hipLaunchKernelGGL(k_count_light<true>, lg, dim3(kLightThreads), lds, s, a, vshift);
    } else {
        hipLaunchKernelGGL(k_count_u<false>, dim3(heavy_wgs), dim3(kThreads), 0, s, a);
        hipLaunchKernelGGL(k_count_light<false>, lg, dim3(kLightThreads), lds, s, a, vshift);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ host side

uint32_t count_wave_span() { return kWaveBits; }
uint32_t count_wave_list(bool per_vertex) { return per_vertex ? kWaveListPV : kSliceWords; }
uint32_t count_block_span() { return kBlockBits; }
uint32_t count_block_list(bool per_vertex) { return per_vertex ? kBlockListPV : kBlockList; }
uint32_t count_item_edges_wave() { return kItemEdgesWave; }
uint32_t count_item_edges_block() { return kItemEdgesBlock; }
uint32_t count_col_pad_bytes() { return kPiece * 4; }
uint32_t count_hcol_pad() { return kPieceHigh - 8; }
uint32_t count_panel() { return kPanel; }
uint32_t count_wgs_per_cu() { return kWgsPerCu; }
uint32_t count_light_max() { return kLightMax; }
uint32_t count_light_chunk_max() { return kLightChunkMax; }
uint32_t count_panel_ranks() { return kPanelRanks; }
uint32_t count_light_list() { return kLightList; }

// Lists per wave: 16, or 8 or 4 where that makes fewer than 16384 waves (16 per SIMD): a wave takes
// its lists' in-edges 64 at a time, one chain of loads after the other.  A resident graph with 16
// lists per wave and by this rule, us: random, 40,000 vertices and 1.3 million edges 152 and 115,
// 200,000 and 12 million 872 and 811; R-MAT, 60,001 and 900,000 91 and 78, 200,003 and 3 million 202
// and 192.  A wave's own cost speaks against it where lists hold one or two in-edges (a wheel of
// 200,000: 22 and 28); a limit of 32768 waves moves the two kinds further apart.
static uint32_t light_shift(uint32_t lists) {
    uint32_t v = kLightShiftMax;
    while (v > kLightShiftMin && (lists >> v) < 16384u) --v;
    return v;
}

hipError_t launch_count(const CountArgs &x, bool per_vertex, hipStream_t s) {
    const dim3 grid(device_cu_count() * kWgsPerCu), block(kThreads);
    if (x.light) {  // before k_count, which adds their totals
        const uint32_t lists = x.lists;
        const uint32_t lshift = light_shift(lists);
        const dim3 lg(ceil_div(lists, kLightWaves << lshift)), lb(kLightThreads);
        if (per_vertex)
            hipLaunchKernelGGL(k_count_light_lists<true>, lg, lb, 0, s, x.row_ptr, x.col, x.cptr,
                               x.cbeg, x.er, lists, x.n1, x.first_panel, x.light, lshift,
                               x.light_total, x.tpv, x.status);
        else
            hipLaunchKernelGGL(k_count_light_lists<false>, lg, lb, 0, s, x.row_ptr, x.col, x.cptr,
                               x.cbeg, x.er, lists, x.n1, x.first_panel, x.light, lshift,
                               x.light_total, x.tpv, x.status);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (per_vertex && x.p0 + 1 < x.n1) {  // panels: those that fit first, on their own queue
        hipLaunchKernelGGL(k_count_panel_pv, grid, block, 0, s, x.row_ptr, x.col, x.cptr,
                           x.cbeg, x.er, x.item_v_b, x.item_off_b,
                           x.n_items_b, x.queue_c, x.total, x.tpv, x.n1, x.first_panel, x.kitem_b,
                           x.hcol, x.hbase, x.status);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (per_vertex)
        hipLaunchKernelGGL(k_count<true>, grid, block, 0, s, x.row_ptr, x.col, x.cptr, x.cbeg,
                           x.er, x.item_v_a, x.item_off_a, x.n_items_a,
                           x.item_v_b, x.item_off_b, x.n_items_b, x.queue_a, x.queue_b, x.total,
                           x.tpv, x.n1, x.first_panel, x.wave_bits, x.block_bits, x.block_list,
                           x.kitem_a, x.kitem_b, x.hcol, x.hrow, x.hbase, x.light_total, x.status);
    else
        hipLaunchKernelGGL(k_count<false>, grid, block, 0, s, x.row_ptr, x.col, x.cptr, x.cbeg,
                           x.er, x.item_v_a, x.item_off_a, x.n_items_a,
                           x.item_v_b, x.item_off_b, x.n_items_b, x.queue_a, x.queue_b, x.total,
                           x.tpv, x.n1, x.first_panel, x.wave_bits, x.block_bits, x.block_list,
                           x.kitem_a, x.kitem_b, x.hcol, x.hrow, x.hbase, x.light_total, x.status);
    return hipGetLastError();
}

}  // namespace tc
