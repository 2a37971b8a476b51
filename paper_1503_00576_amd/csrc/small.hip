// Preprocessing steps for small graphs (at most kSmallVertices vertices and kSmallEntries entries
// of the edge array): the same arrays as the general path, in fewer launches.
//
// A count of a small graph is bound by its launches, 4 to 15 us each whatever they do: the general
// path takes four for the degrees, two to four for the order, five or six for the edge sort and
// as many for the in-edge lists, since its partitions and radix passes are made for arrays that
// fit no cache.  Here every vertex has a counter in one workgroup's LDS and every array stays in
// L2, so the degrees are one launch, the order is one (each vertex counts the keys below its
// own), and both sorts are counting sorts: a position inside the row (list) from an atomic when
// the entry is formed, and a placement once the rows' offsets are scanned.  The order inside a
// row is then settled by the row sort; inside a list it does not matter.  18 launches instead of
// 30: a count of 8,009 vertices and 100,003 edges took 221 us and takes 132, one of G(1000, 0.02)
// 219 and 111.  The limits are those of the LDS counters (64 KB) and of the atomics: the order
// grows with the square of the vertices (17 us at 8,009), the placement with the entries (20 us
// at 100,003), where the general path's steps hardly grow.
#include "internal.h"

namespace tc {

constexpr uint32_t kSmallVertices = 16384;
constexpr uint32_t kSmallEntries = 1u << 18;
constexpr uint32_t kSmallTile = 4096;  // entries per workgroup of 1024 threads

uint32_t small_vertices() { return kSmallVertices; }
uint32_t small_entries() { return kSmallEntries; }

// degrees and the checks of the input: counters of all vertices in LDS, added to deg once per
// workgroup and vertex
__global__ __launch_bounds__(1024) void k_s_degree(const int2 *__restrict__ edges, uint32_t m,
                                                   uint32_t n, uint32_t both,
                                                   uint32_t *__restrict__ deg,
                                                   int32_t *__restrict__ status) {
    __shared__ uint32_t cnt[kSmallVertices];
    const uint32_t t = threadIdx.x;
    int2 e[kSmallTile / 1024];
#pragma unroll
    for (uint32_t k = 0; k < kSmallTile / 1024; ++k) {
        const uint32_t i = blockIdx.x * kSmallTile + k * 1024 + t;
        e[k] = i < m ? edges[i] : make_int2(0, 0);
    }
    for (uint32_t i = t; i < n; i += 1024) cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kSmallTile / 1024; ++k) {
        const uint32_t i = blockIdx.x * kSmallTile + k * 1024 + t;
        if (i >= m) continue;
        if ((uint32_t)e[k].x >= n || (uint32_t)e[k].y >= n) {
            set_status(status, TC_E_RANGE);
        } else if (e[k].x == e[k].y) {
            set_status(status, TC_E_SELF_LOOP);
        } else {
            atomicAdd(&cnt[e[k].x], 1u);
            if (!both) atomicAdd(&cnt[e[k].y], 1u);
        }
    }
    __syncthreads();
    for (uint32_t i = t; i < n; i += 1024)
        if (cnt[i]) atomicAdd(&deg[i], cnt[i]);
}

// The order of Section 2.2: rank[v] = number of vertices with a smaller (degree, id).  64 vertices
// per workgroup, one per lane; every wave compares them with its sixteenth of all keys, four
// at a time from LDS (the same ones for all lanes).
__global__ __launch_bounds__(1024) void k_s_rank(const uint32_t *__restrict__ deg, uint32_t n,
                                                 uint32_t *__restrict__ perm,
                                                 uint32_t *__restrict__ rank,
                                                 const int32_t *__restrict__ status) {
    __shared__ __align__(16) uint32_t key[kSmallVertices];
    __shared__ uint32_t below[kWave];
    if (*status) return;
    const uint32_t t = threadIdx.x, lane = lane_id(), w = t / kWave;
    // (degree, id) in 32 bits: ids below 2^14, degrees below 2^14 in a simple graph (cut off at
    // 2^18 - 1, which only repeated edges reach)
    const uint32_t n4 = (n + 3u) & ~3u;
    for (uint32_t i = t; i < n4; i += 1024)
        key[i] = i < n ? (min(deg[i], (1u << 18) - 1u) << 14) | i : ~0u;
    if (t < kWave) below[t] = 0;
    __syncthreads();
    const uint32_t v = blockIdx.x * kWave + lane;
    const uint32_t mine = v < n ? key[v] : 0u;
    const uint32_t quads = n4 / 4, q0 = quads * w / 16, q1 = quads * (w + 1) / 16;
    uint32_t c = 0;
    for (uint32_t q = q0; q < q1; ++q) {
        const uint4 k = reinterpret_cast<const uint4 *>(key)[q];
        c += (k.x < mine) + (k.y < mine) + (k.z < mine) + (k.w < mine);
    }
    atomicAdd(&below[lane], c);
    __syncthreads();
    if (w == 0 && v < n) {
        rank[v] = below[lane];
        perm[below[lane]] = v;
    }
}

// every kept edge as (source << 16 | target, position inside its row), all ones for a dropped entry
// of the two-direction format, whose forward entries are counted; re[s] = entries of row s
__global__ __launch_bounds__(256) void k_s_orient(const int2 *__restrict__ edges, uint32_t m,
                                                  uint32_t both,
                                                  const uint32_t *__restrict__ rank,
                                                  uint32_t *__restrict__ re,
                                                  uint2 *__restrict__ out,
                                                  uint32_t *__restrict__ counter,
                                                  const int32_t *__restrict__ status) {
    __shared__ uint32_t s_cnt[4];
    if (*status) return;
    const uint32_t t = threadIdx.x;
    uint32_t kept = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t i = blockIdx.x * 1024 + k * 256 + t;
        bool keep = false;
        if (i < m) {
            const int2 e = edges[i];
            const uint32_t ru = rank[e.x], rv = rank[e.y];
            keep = !both || ru < rv;
            uint2 x = make_uint2(~0u, 0u);
            if (keep) {
                const uint32_t s = min(ru, rv);
                x = make_uint2((s << 16) | max(ru, rv), atomicAdd(&re[s], 1u));
            }
            out[i] = x;
        }
        kept += (uint32_t)__popcll(__ballot(keep));
    }
    if (!both) return;
    if (lane_id() == 0) s_cnt[t / kWave] = kept;
    __syncthreads();
    if (t == 0) atomicAdd(counter, s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3]);
}

// neighbour and source arrays (rows in any order), and rchunk[c] = the first row that starts at or
// after position c * chunk
__global__ __launch_bounds__(256) void k_s_place(const uint2 *__restrict__ in, uint32_t m,
                                                 uint32_t both, uint32_t mf, uint32_t chunk,
                                                 const uint32_t *__restrict__ row_ptr,
                                                 const uint32_t *__restrict__ counter,
                                                 uint32_t *__restrict__ col,
                                                 uint32_t *__restrict__ src,
                                                 uint32_t *__restrict__ rchunk,
                                                 int32_t *__restrict__ status) {
    if (*status) return;
    if (both && *counter != mf) {  // exactly half of the entries must be forward
        if (threadIdx.x == 0) set_status(status, TC_E_ASYMMETRIC);
        return;
    }
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const uint2 x = in[i];
    if (x.x == ~0u) return;
    const uint32_t s = x.x >> 16, pos = row_ptr[s] + x.y;
    col[pos] = x.x & 0xFFFFu;
    src[pos] = s;
    if (pos % chunk == 0) rchunk[pos / chunk] = x.y == 0 ? s : s + 1;
}

// Position of every listed in-edge inside its list (cid[e] its list, `lists` and more for none):
// a workgroup counts its entries per list in LDS and claims their room in each list with one
// atomic on lre[list], so that the panels' long lists, which most workgroups meet, do not queue.
__global__ __launch_bounds__(1024) void k_s_lists(const uint32_t *__restrict__ cid, uint32_t mf,
                                                  uint32_t lists, uint32_t *__restrict__ lre,
                                                  uint32_t *__restrict__ pos,
                                                  const int32_t *__restrict__ status) {
    __shared__ uint32_t cnt[kSmallVertices + 1];
    if (*status) return;
    const uint32_t t = threadIdx.x;
    constexpr uint32_t kPer = kSmallTile / 1024;
    uint32_t c[kPer], at[kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t e = blockIdx.x * kSmallTile + k * 1024 + t;
        c[k] = e < mf ? cid[e] : lists;
        at[k] = ~0u;
    }
    for (uint32_t i = t; i < lists; i += 1024) cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
        if (c[k] < lists) at[k] = atomicAdd(&cnt[c[k]], 1u);
    __syncthreads();
    // (one entry of each list is its first in this workgroup)
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
        if (at[k] == 0) cnt[c[k]] = atomicAdd(&lre[c[k]], cnt[c[k]]);
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t e = blockIdx.x * kSmallTile + k * 1024 + t;
        if (c[k] < lists) pos[e] = cnt[c[k]] + at[k];
    }
}

__global__ __launch_bounds__(256) void k_s_place_lists(const uint32_t *__restrict__ cid,
                                                       const uint32_t *__restrict__ pos,
                                                       uint32_t mf, uint32_t lists,
                                                       const uint32_t *__restrict__ cptr,
                                                       uint32_t *__restrict__ cbeg,
                                                       const int32_t *__restrict__ status) {
    if (*status) return;
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= mf) return;
    const uint32_t c = cid[e];
    if (c < lists) cbeg[cptr[c] + pos[e]] = e + 1;
}

hipError_t small_order(const int32_t *edges, uint32_t m, uint32_t n, bool both, uint32_t *deg,
                       uint32_t *perm, uint32_t *rank, int32_t *status, hipStream_t s) {
    hipLaunchKernelGGL(k_s_degree, dim3(ceil_div(m, kSmallTile)), dim3(1024), 0, s,
                       (const int2 *)edges, m, n, (uint32_t)both, deg, status);
    hipLaunchKernelGGL(k_s_rank, dim3(ceil_div(n, kWave)), dim3(1024), 0, s, deg, n, perm, rank,
                       status);
    return hipGetLastError();
}

hipError_t small_rows(const int32_t *edges, uint32_t m, uint32_t n, bool both, uint32_t mf,
                      const uint32_t *rank, uint2 *tmp, const uint32_t *rs, uint32_t *re,
                      uint32_t *row_ptr, uint32_t *col, uint32_t *src, uint32_t *rchunk,
                      uint32_t *counter, uint32_t *scan_scratch, int32_t *status, hipStream_t s) {
    hipLaunchKernelGGL(k_s_orient, dim3(ceil_div(m, 1024)), dim3(256), 0, s, (const int2 *)edges,
                       m, (uint32_t)both, rank, re, tmp, counter, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = scan_row_bounds(rs, re, n, row_ptr, scan_scratch, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_s_place, dim3(ceil_div(m, 256)), dim3(256), 0, s, tmp, m, (uint32_t)both,
                       mf, row_sort_chunk(mf), row_ptr, counter, col, src, rchunk, status);
    return hipGetLastError();
}

hipError_t small_lists(const uint32_t *cid, uint32_t mf, uint32_t lists, const uint32_t *lrs,
                       uint32_t *lre, uint32_t *pos, uint32_t *cptr, uint32_t *cbeg,
                       uint32_t *scan_scratch, int32_t *status, hipStream_t s) {
    hipLaunchKernelGGL(k_s_lists, dim3(ceil_div(mf, kSmallTile)), dim3(1024), 0, s, cid, mf, lists,
                       lre, pos, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = scan_row_bounds(lrs, lre, lists, cptr, scan_scratch, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_s_place_lists, dim3(ceil_div(mf, 256)), dim3(256), 0, s, cid, pos, mf,
                       lists, cptr, cbeg, status);
    return hipGetLastError();
}

}  // namespace tc
